// The two score passes (score.hip) in float32, the mode that checks the 16-bit one.
//
// A float32 product costs sixteen times the matrix time of a 16-bit one.  Every operand is therefore
// written as the exact sum of three bf16 pieces (a float's 24 digits are three times eight),
// x = h + m + l with |m| <= 2^-9 |x|, |l| <= 2^-18 |x|, and a product as the six products of pieces down to
// 2^-18: hh, hm, mh, mm, hl, lh (what is left out, ml, lm and ll, is below 2^-26 of it); the method is that of Henry, Tang and Heinecke,
// "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", ARITH 2019.  Six
// 32x32x16 instructions of 32 clocks stand where eight 32x32x2 ones of 64 did.  Those with a lower piece are summed first, over all
// columns, those of the high pieces last: a sum of 128 products is rounded 8 times at its full size instead of 64 times.
// Measured (us of the first / second pass by float32 products, now): 8 heads over 2 of 128, 3000 rows
// 93.5 / 107.1 -> 54.7 / 62.5; 32 over 8, 6000 rows 1242 / 1279 -> 702 / 718, of 64 594 / 604 -> 394 / 394; the whole case of 8 heads
// 226 -> 141.  Errors against 64 bits, by float32 products / column by column / now: row log-sum-exp, rms, 3000 rows
// of 128 7.7e-7 / 6.7e-7 / 4.6e-7, of 64 7.0e-7 / 6.1e-7 / 4.6e-7.  Column sums, 2-norm of the error over that of the sums, means of 12 to 48 seeds of 13 shapes of 600 to 6000
// rows, each below its own figure by float32 products: of 128 0.9-2.1e-7 -> 0.7-1.3e-7 (all rows), 1.2-2.7e-7 -> 0.8-1.4e-7 (window), of 64 0.7-1.6e-7 -> 0.6-0.8e-7,
// 1.2-2.1e-7 -> 0.8-1.1e-7.  With every column weighted alike, whatever its sum, 0.9-1.8e-7 -> 0.8-1.0e-7 of 128, but of 64 1.0-1.5e-7 -> 1.2-1.4e-7 (window
// 1.2-2.0e-7 -> 1.4-1.7e-7): the 16-bit matrix instruction's own sums draw the logits towards zero by 4e-9 of their size, which lifts the smallest weights.
//
// A wave keeps 64 rows in registers as their pieces (split once per item) and streams the other operand as
// float32 through its ring of two stages; a stage is split on the way to the matrix pipe, in the vector slots
// between the products: per 16 columns 12 products (384 clocks), 44 operations of splitting, 12 to 24 of weighing the
// stage before (beside the products of the high pieces, where there is nothing to split, as much of that as fits).  That is what bounds it: 3072 clocks of products and up to 2900 of issue per stage of 32 x 64 x 128.
//
// Not every float has three such pieces.  Infinities, NaN and values that round to infinity in bf16 give NaN, which no
// later step loses; rows with elements of 2^60 and more, or below 2^-100 (whose low piece falls below bf16's range
// while the other factor could be large), are found when they are split.  The latter's items go by float32 products, of any values, from the
// first stage on; the others' from the set of stages on whose sums left the float range (they are put back to what they were before it), so that
// infinite logits come out as by float32 products, at about their cost.  One key of -inf, which every later row of its head streams, us
// of both passes by float32 products alone / begun anew without a pipeline / now: 8 heads over 2 of 128, 3000 rows 235 / 315 / 212, of 64 113 / 168 / 116;
// 32 over 8, 6000 rows 3361 / 4197 / 2576; 4 x 32 over 8, 4096 4690 / 7922 / 5034 (a wave alone at that pace, among others that draw
// the power of 16-bit products), in the middle of the sequence 4929 / - / 3394; a large element in every key 4701 / 6376 / 3556.
#include "ems_common.h"
#include "ems_kernels.h"
#include "ems_score.h"
#include "ems_stream.h"

namespace ems {

// Stages from one look at the sums to the next: two, and twice as many each time up to this.  (What the first value without pieces
// throws away is then little against what went well before it.)
constexpr int kFoldStagesF32 = 8;

typedef __bf16 bf16x2v_t __attribute__((ext_vector_type(2)));
typedef float f32x2v_t __attribute__((ext_vector_type(2)));

// two floats -> their bf16 pieces of one level (rounded to nearest even), and what they leave
__device__ __forceinline__ int split_pair(float& x0, float& x1)
{
    const int p = __builtin_bit_cast(int, __builtin_convertvector(f32x2v_t{x0, x1}, bf16x2v_t));
    x0 -= __builtin_bit_cast(float, p << 16);
    x1 -= __builtin_bit_cast(float, p & (int)0xffff0000);
    return p;
}
__device__ __forceinline__ int last_pair(float x0, float x1)
{
    return __builtin_bit_cast(int, __builtin_convertvector(f32x2v_t{x0, x1}, bf16x2v_t));
}

// Eight consecutive-in-K elements of a row as pieces: the operand of three products.
struct Pieces { frag_t h, m, l; };

__device__ __forceinline__ void mma_piece(f32x16_t& acc, const frag_t& a, const frag_t& b, bool start)
{
    if (start) mma_first<bf16_t>(acc, a, b);
    else mma<bf16_t>(acc, a, b);
}

// Keeps what forms the value before this point (the compiler would move a stage's vector work past its
// last product, where branches follow and the matrix pipe is idle).
__device__ __forceinline__ void stays_here(float& x) { asm volatile("" : "+v"(x)); }

template <int D>
struct F32 {
    static constexpr int kFrags = Tile<float, D>::kFrags;              // 16-byte fragments a lane has of a row
    static constexpr int kSteps = kFrags / 2;                          // 16 columns each
    static constexpr int kRowBytes = Tile<float, D>::kRowBytes;
    static constexpr int kCpr = Tile<float, D>::kChunksPerRow;
    static constexpr int kStageBytes = kStreamRows * kRowBytes;
    static constexpr int kInstr = kStageBytes / 1024;                  // DMA instructions per stage
    static_assert(kInstr % 4 == 0 && kSteps % 2 == 0 && kSteps >= 4, "");

    // where a lane finds its fragments of its row of 32, 32 bytes apart (past the end of the matrix: of the last row, whose
    // results there are not kept)
    static __device__ __forceinline__ const char* row_bytes(const float* X, int row0, int N, int lane)
    {
        return reinterpret_cast<const char*>(X) + (size_t)min(row0 + (lane & 31), N - 1) * kRowBytes + (lane >> 5) * 16;
    }
    // the 32 * kSubF32 rows from row0 on, as pieces; true if a row's elements may not be split (see above)
    static __device__ __forceinline__ bool load_stationary(const float* X, int row0, int N, int lane, Pieces (&b)[kSubF32][kSteps])
    {
        float most = 0.f, least = INFINITY;
#pragma unroll
        for (int s = 0; s < kSubF32; ++s) {
            const char* x = row_bytes(X, row0 + s * 32, N, lane);
            frag_t raw[kFrags];
#pragma unroll
            for (int f = 0; f < kFrags; ++f) raw[f] = *reinterpret_cast<const frag_t*>(x + f * 32);
#pragma unroll
            for (int f = 0; f < kSteps; ++f) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const f32x4_t v = __builtin_bit_cast(f32x4_t, raw[2 * f + w / 2]);
                    float x0 = v[2 * (w & 1)], x1 = v[2 * (w & 1) + 1];
                    most = fmaxf(most, fmaxf(fabsf(x0), fabsf(x1)));
                    least = fminf(least, fminf(x0 == 0.f ? INFINITY : fabsf(x0), x1 == 0.f ? INFINITY : fabsf(x1)));
                    b[s][f].h[w] = split_pair(x0, x1);
                    b[s][f].m[w] = split_pair(x0, x1);
                    b[s][f].l[w] = last_pair(x0, x1);
                }
                // (the accumulation registers, which only the products read)
                asm volatile("" : "+a"(b[s][f].h)); asm volatile("" : "+a"(b[s][f].m)); asm volatile("" : "+a"(b[s][f].l));
            }
            __builtin_amdgcn_sched_barrier(0);                         // one subtile's rows at a time
        }
        return !(most < 0x1p60f) || least < 0x1p-100f;
    }

    // the same rows as they are
    static __device__ __forceinline__ void load_exact(const float* X, int row0, int N, int lane, frag_t (&b)[kSubF32][kFrags])
    {
#pragma unroll
        for (int s = 0; s < kSubF32; ++s) {
            const char* x = row_bytes(X, row0 + s * 32, N, lane);
#pragma unroll
            for (int f = 0; f < kFrags; ++f) b[s][f] = *reinterpret_cast<const frag_t*>(x + f * 32);
        }
#pragma unroll
        for (int s = 0; s < kSubF32; ++s)
#pragma unroll
            for (int f = 0; f < kFrags; ++f) asm volatile("" : "+a"(b[s][f]));
    }

    // Source offsets of a stage's DMA, less what the instruction itself adds (1 KiB x its place in a group of four); those of
    // the stage's second 16 rows are the same again.
    static constexpr int kOffs = kInstr / 2;
    static_assert(kOffs % 4 == 0, "");
    static __device__ __forceinline__ void dma_offsets(int lane, unsigned (&off)[kOffs])
    {
#pragma unroll
        for (int j = 0; j < kOffs; ++j) {
            const int slot = j * kWave + lane, row = slot / kCpr;
            off[j] = (unsigned)row * kRowBytes + (unsigned)(((slot % kCpr) ^ swz_key<float, D>(row)) << 4) - (unsigned)(j % 4) * 1024u;
        }
    }
    // DMA of 32 rows from `row` on into the ring slot at `dst`; rows past the end re-read the last one
    static __device__ __forceinline__ void issue(const char* base, int row, int N, unsigned dst, const unsigned (&off)[kOffs])
    {
        const char* from = base + (size_t)row * kRowBytes;
        if (row + kStreamRows <= N) {
#pragma unroll
            for (int j = 0; j < kInstr; j += 4) {
                const int i = j % kOffs;
                dma_to_lds_x4(from + j / kOffs * (16 * kRowBytes), off[i], off[i + 1], off[i + 2], off[i + 3], dst + j * 1024);
            }
        } else {
            const int lane = lane_here();                              // (nothing is kept for this)
#pragma unroll
            for (int j = 0; j < kInstr; ++j) {
                const int over = max(row + (j * kWave + lane) / kCpr - (N - 1), 0);
                dma_to_lds<16>(base, (unsigned)row * kRowBytes + off[j % kOffs] + j / kOffs * (16 * kRowBytes) + (unsigned)(j % 4) * 1024u - (unsigned)over * kRowBytes, dst + j * 1024);
            }
        }
    }
    // a lane's fragment f of its row of a stage (the swizzle touches the low chunk bits only)
    static constexpr int kKeys = kCpr >= 16 ? 8 : 4;                   // distinct offsets: 16 or 8 chunks swizzled together, two of a fragment
    static __device__ __forceinline__ void frag_offsets(int lane, unsigned (&off)[kKeys])
    {
        const int col = lane & 31, half = lane >> 5;
#pragma unroll
        for (int f = 0; f < kKeys; ++f) off[f] = (unsigned)col * kRowBytes + (unsigned)(((f * 2 + half) ^ swz_key<float, D>(col)) << 4);
    }
    static __device__ __forceinline__ frag_t fetch(const char* stage, const unsigned (&off)[kKeys], int f)
    {
        return *reinterpret_cast<const frag_t*>(stage + off[f % kKeys] + (f / kKeys) * (kKeys * 32));
    }

    // The streamed operand on its way from LDS to the matrix pipe: raw fragments two steps ahead of the products,
    // pieces one.
    struct Feed {
        frag_t raw[2][2];                                              // by step parity
        Pieces now, next;
        float x[8];                                                    // what is left of the elements being split
        __device__ __forceinline__ void take(int parity)
        {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const f32x4_t v = __builtin_bit_cast(f32x4_t, raw[parity][i]);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[4 * i + e] = v[e];
            }
        }
        __device__ __forceinline__ void part(int slot)                 // 1/10 of the splitting
        {
            if (slot < 4) next.h[slot] = split_pair(x[2 * slot], x[2 * slot + 1]);
            else if (slot < 8) next.m[slot - 4] = split_pair(x[2 * slot - 8], x[2 * slot - 7]);
            else {
#pragma unroll
                for (int w = 2 * slot - 16; w < 2 * slot - 14; ++w) next.l[w] = last_pair(x[2 * w], x[2 * w + 1]);
            }
        }
        // the first step of the first stage
        __device__ __forceinline__ void start(const char* stage, const unsigned (&off)[kKeys])
        {
            raw[0][0] = fetch(stage, off, 0); raw[0][1] = fetch(stage, off, 1);
            raw[1][0] = fetch(stage, off, 2); raw[1][1] = fetch(stage, off, 3);
            take(0);
#pragma unroll
            for (int k = 0; k < kLow; ++k) part(k);
            now = next;
        }
    };

    // The products of one stage, 32 streamed rows x kSubF32 tiles; the two tiles' chains alternate.  Those with a lower piece come first, step by
    // step, then those of the high pieces, so that only the latter are rounded at the size of the whole sum.  `landed` waits for the next stage
    // (which step kSteps - 2 begins to read); `begin(s)`: vector work ahead of tile s's; `weigh(e)`: vector work of element e of 2 * 16, in
    // the slots that the splitting leaves room in.
    static constexpr int kLow = 10, kEach = 32 / kSteps - 2;           // slots of a step; elements weighed in its last ones, the rest beside the high pieces
    template <class Landed, class Begin, class Weigh>
    static __device__ __forceinline__ void stage(const char* here, const char* after, const unsigned (&off)[kKeys], Feed& q,
                                                 const Pieces (&b)[kSubF32][kSteps], f32x16_t (&acc)[kSubF32], Landed landed, Begin begin, Weigh weigh)
    {
        frag_t high[kSteps];
#pragma unroll
        for (int f = 0; f < kSteps; ++f) {
            if (f == kSteps - 2) landed();
            q.take((f + 1) & 1);
            {
                const char* from = f + 2 < kSteps ? here : after;
                const int at = (f + 2) % kSteps * 2;
                q.raw[f & 1][0] = fetch(from, off, at);
                q.raw[f & 1][1] = fetch(from, off, at + 1);
            }
            high[f] = q.now.h;
            asm volatile("" : "+a"(high[f]));                          // (only the products read it)
#pragma unroll
            for (int i = 0; i < kLow; ++i) {
                const int s = i & 1, k = i >> 1;
                const Pieces& p = b[s][f];
                const frag_t& x = k == 0 ? q.now.l : k == 1 || k == 3 ? high[f] : q.now.m;
                const frag_t& y = k == 1 ? p.l : k == 2 || k == 3 ? p.m : p.h;
                mma_piece(acc[s], x, y, f == 0 && k == 0);
                q.part(i);
                if (f == 0 && i < kSubF32) begin(i);
                if (i >= kLow - kEach) weigh(f * kEach + i - (kLow - kEach));
                __builtin_amdgcn_sched_barrier(0);
            }
            q.now = q.next;
        }
        asm volatile("" : "+v"(q.now.h)); asm volatile("" : "+v"(q.now.m)); asm volatile("" : "+v"(q.now.l));       // (as in stays_here)
#pragma unroll
        for (int i = 0; i < 2 * kSteps; ++i) {
            mma<bf16_t>(acc[i & 1], high[i >> 1], b[i & 1][i >> 1].h);
            weigh(kSteps * kEach + i);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // The same by float32 products, of any values.  `first`: a lane's first fragment, fetched a stage ahead; `early`: what waits for nothing.
    template <class Early, class Landed, class Begin, class Weigh>
    static __device__ __forceinline__ void exact_stage(const char* here, const char* after, const unsigned (&off)[kKeys], frag_t& first,
                                                       const frag_t (&b)[kSubF32][kFrags], f32x16_t (&acc)[kSubF32], Early early, Landed landed,
                                                       Begin begin, Weigh weigh)
    {
        frag_t x[2];
        x[0] = first;
#pragma unroll
        for (int f = 0; f < kFrags; ++f) {
            if (f + 1 < kFrags) x[(f + 1) & 1] = fetch(here, off, f + 1);
            else { landed(); first = fetch(after, off, 0); }
#pragma unroll
            for (int s = 0; s < kSubF32; ++s) {
                if (f == 0) mma_first<float>(acc[s], x[0], b[s][0]);
                else mma<float>(acc[s], x[f & 1], b[s][f]);
                if (f == 0 && s == 0) { begin(0); begin(1); }
                if (f == 0 && s == 1) early();
#pragma unroll
                for (int e = (2 * f + s) * 16 / kFrags; e < (2 * f + s + 1) * 16 / kFrags; ++e) weigh(e);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
};

// ------------------------------------------------------------------------------------
// Second pass: 64 keys stationary, the query rows of every q-head of the group streamed with their log-sum-exp.
// The weights of a stage are formed under the products of the next one; those of a stage with window rows (which go
// to the local sums too), and by float32 products of one on the diagonal, at its end.  By pieces rows above the diagonal get logits of -inf.
// ------------------------------------------------------------------------------------
template <int D, bool kDeal>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(1, 1))) void score_pass2_f32_kernel(ScoreArgs a)
{
    using E = F32<D>;
    constexpr int kSub = kSubF32, kKeys = 32 * kSub;
    __shared__ __attribute__((aligned(1024))) char lds_q[2][E::kStageBytes];
    __shared__ __attribute__((aligned(256))) float lds_lse[2][2 * kStreamRows];       // second half: spare

    const float c = a.scale_log2e;
    const int N = a.seq_len, win0 = N - a.window, G = a.q_heads / a.kv_heads;
    Pass2Items<kSub, kDeal> items(a);
    while (items.next()) {
    const int key_base = items.J * kKeys, bkv = items.bkv, r_begin = items.r_begin, r_end = items.r_end;
    const int b = bkv / a.kv_heads, kvh = bkv % a.kv_heads;
    const float* K = reinterpret_cast<const float*>(a.k) + ((size_t)bkv * N) * D;
    const float* Q0 = reinterpret_cast<const float*>(a.q) + ((size_t)(b * a.q_heads + kvh * G) * N) * D;
    const float* L0 = a.lse2 + (size_t)(b * a.q_heads + kvh * G) * a.n_pad;
    const int lane = opaque_lane(threadIdx.x);
    const int col = lane & 31, half = lane >> 5;

    unsigned dma_off[E::kOffs], frag_off[E::kKeys];
    E::dma_offsets(lane, dma_off);
    E::frag_offsets(lane, frag_off);
    const unsigned lds_q0 = lds_address(&lds_q[0][0]), lds_l0 = lds_address(&lds_lse[0][0]);

    const int per_head = (r_end - r_begin + kStreamRows - 1) / kStreamRows, n_stages = per_head * G;
    float glo[kSub], loc[kSub];
#pragma unroll
    for (int s = 0; s < kSub; ++s) glo[s] = loc[s] = 0.f;

    // Stages [from, n_stages).  kExact: by float32 products.  By pieces: up to a set of stages that leaves a sum out of the float range; the sums are then
    // as before it.  Returns the first stage that is not in the sums.
    auto sweep = [&](auto exact_c, const auto& bk, int from) __attribute__((always_inline)) {
        constexpr bool kExact = decltype(exact_c)::value;
        int g_next = scalar(from / per_head), row_next = r_begin + (from - g_next * per_head) * kStreamRows;      // the stage to fetch next
        int row_now = row_next;
        auto issue_next = [&](int slot) __attribute__((always_inline)) {
            E::issue(reinterpret_cast<const char*>(Q0) + (size_t)g_next * N * E::kRowBytes, row_next, N, lds_q0 + slot * E::kStageBytes, dma_off);
            // the rows' log-sum-exp (+inf up to n_pad); the upper half-wave's copy goes to the spare half of the slot
            dma_to_lds<4>(L0 + (size_t)g_next * a.n_pad, (unsigned)(row_next + col) * 4u, lds_l0 + slot * (2 * kStreamRows * 4));
            row_next += kStreamRows;
            if (row_next >= r_end) { row_next = r_begin; ++g_next; }
        };

        f32x16_t acc[2][kSub], lse_v[2];
        float part[kSub][2], glo_in[kSub], loc_in[kSub];
        bool counted = false;                                           // the last stage's weights are in the sums
#pragma unroll
        for (int s = 0; s < kSub; ++s) { part[s][0] = part[s][1] = 0.f; glo_in[s] = glo[s]; loc_in[s] = loc[s]; acc[1][s] = zero_acc(); }
#pragma unroll
        for (int r = 0; r < 16; ++r) lse_v[1][r] = INFINITY;            // before the first stage: weights of zero
        typename E::Feed feed;
        frag_t first = zero_frag();
        wait_lds_all_visible();
        issue_next(0);
        wait_vmem<0>();
        if constexpr (kExact) first = E::fetch(lds_q[0], frag_off, 0);
        else feed.start(lds_q[0], frag_off);

        auto stage = [&](auto set_c, int t) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            // the other slot was last read (its log-sum-exp included) before the last steps of the stage before this one
            auto issue = [&]() __attribute__((always_inline)) { wait_lds_all_visible(); if (t + 1 < n_stages) issue_next(1 - set); };
            auto landed = []() __attribute__((always_inline)) { wait_vmem<0>(); };
            if constexpr (!kExact) issue();
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const f32x4_t v = *reinterpret_cast<const f32x4_t*>(lds_lse[set] + 8 * q4 + 4 * half);
#pragma unroll
                for (int i = 0; i < 4; ++i) lse_v[set][4 * q4 + i] = v[i];
            }
            auto weigh = [&](int e) __attribute__((always_inline)) {    // (of the stage before)
                const int s = e & 1, r = e >> 1;
                part[s][r & 1] += exp2_fast(__builtin_fmaf(acc[1 - set][s][r], c, -lse_v[1 - set][r]));
            };
            if constexpr (kExact) {
                E::exact_stage(lds_q[set], lds_q[1 - set], frag_off, first, bk, acc[set], issue, landed, [](int) __attribute__((always_inline)) {}, weigh);
            } else {
                E::stage(lds_q[set], lds_q[1 - set], frag_off, feed, bk, acc[set], landed, [](int) __attribute__((always_inline)) {}, weigh);
            }
#pragma unroll
            for (int s = 0; s < kSub; ++s) { stays_here(part[s][0]); stays_here(part[s][1]); }
            const int row0 = row_now;
            row_now += kStreamRows;
            if (row_now >= r_end) row_now = r_begin;
            const bool diagonal = row0 < key_base + kKeys;              // rows before the key are above it
            counted = row0 + kStreamRows > win0 || (kExact && diagonal);
            if (!kExact && diagonal) {
                const int lane = lane_here(), col = lane & 31, half = lane >> 5;      // (nothing is kept for this)
#pragma unroll
                for (int s = 0; s < kSub; ++s)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (row0 + acc_row(r, half) < key_base + s * 32 + col) acc[set][s][r] = -INFINITY;
            }
            if (counted) {                                              // at once, and none left for the next stage
                const int lane = lane_here(), col = lane & 31, half = lane >> 5;
#pragma unroll
                for (int s = 0; s < kSub; ++s) {
                    float p[16];
#pragma unroll
                    for (int r = 0; r < 16; ++r) p[r] = exp2_fast(__builtin_fmaf(acc[set][s][r], c, -lse_v[set][r]));
                    // (above the diagonal no weight, whatever the log-sum-exp: minus infinity would make NaN of a logit of minus infinity)
                    if (kExact) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) p[r] = row0 + acc_row(r, half) < key_base + s * 32 + col ? 0.f : p[r];
                    }
                    part[s][0] += sum16(p);
#pragma unroll
                    for (int r = 0; r < 16; ++r) p[r] = row0 + acc_row(r, half) < win0 ? 0.f : p[r];
                    loc[s] += sum16(p);
                    acc[set][s] = zero_acc();
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) lse_v[set][r] = INFINITY;
            }
        };
        // the sums so far are set aside; by pieces, they are those before the set again where one of them has left the float range
        auto fold = [&]() __attribute__((always_inline)) {
            bool left = false;
#pragma unroll
            for (int s = 0; s < kSub; ++s) {
                glo[s] += part[s][0] + part[s][1];
                part[s][0] = part[s][1] = 0.f;
                left |= (glo_in[s] < INFINITY && !(glo[s] < INFINITY)) || (loc_in[s] < INFINITY && !(loc[s] < INFINITY));
            }
            if constexpr (kExact) return false;
            const bool any = __any(left);                               // wave-uniform
#pragma unroll
            for (int s = 0; s < kSub; ++s) {
                if (any) { glo[s] = glo_in[s]; loc[s] = loc_in[s]; }
                else { glo_in[s] = glo[s]; loc_in[s] = loc[s]; }
            }
            return any;
        };
        int run = 2, until_fold = run;
        int t = from;
        do {                                                            // (an item has rows)
            stage(ic<0>{}, t);
            if (t + 1 < n_stages) stage(ic<1>{}, t + 1);
            until_fold -= 2;
            if (until_fold <= 0 && t + 2 < n_stages) {
                until_fold = run = min(2 * run, kFoldStagesF32);
                if (fold()) return from;
                from = counted ? t + 2 : t + 1;
            }
        } while ((t += 2) < n_stages);
        wait_vmem<0>();
        auto last = [&](const f32x16_t (&x)[kSub], const f32x16_t& l) __attribute__((always_inline)) {
#pragma unroll
            for (int s = 0; s < kSub; ++s)
#pragma unroll
                for (int r = 0; r < 16; ++r) part[s][r & 1] += exp2_fast(__builtin_fmaf(x[s][r], c, -l[r]));
        };
        if ((t - n_stages) & 1) last(acc[0], lse_v[0]);
        else last(acc[1], lse_v[1]);
        return fold() ? from : n_stages;
    };
    int from = 0;
    {
        Pieces bk[kSub][E::kSteps];
        const bool whole = !__any(E::load_stationary(K, key_base, N, lane, bk));
        wait_vmem_all_visible();
        if (whole) from = scalar(sweep(std::false_type{}, bk, 0));
    }
    if (from < n_stages) {
        frag_t bk[kSub][E::kFrags];
        E::load_exact(K, key_base, N, lane, bk);
        wait_vmem_all_visible();
        sweep(std::true_type{}, bk, from);
    }
    float *out_glo, *out_loc;
    items.outputs(out_glo, out_loc);
#pragma unroll
    for (int s = 0; s < kSub; ++s) {
        const float gsum = halves_sum(glo[s]), lsum = halves_sum(loc[s]);         // the half-waves hold disjoint rows of the same keys
        const int kj = key_base + s * 32 + col;
        if (half == 0 && kj < N) {
            out_glo[kj] = gsum;
            if (out_loc) out_loc[kj] = lsum;
        }
    }
    }   // next work item
}

// ------------------------------------------------------------------------------------
// First pass: 64 query rows stationary, keys streamed.  The running maximum and the rescaled sum of a stage are formed under the
// products of the next one; keys above the diagonal get logits of -inf.
// ------------------------------------------------------------------------------------
template <int D, bool kDeal>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(1, 1))) void score_pass1_f32_kernel(ScoreArgs a)
{
    using E = F32<D>;
    constexpr int kSub = kSubF32, kRows = 32 * kSub;
    __shared__ __attribute__((aligned(1024))) char lds_k[2][E::kStageBytes];

    const float c = a.scale_log2e;
    const int N = a.seq_len, G = a.q_heads / a.kv_heads;
    Pass1Items<kSub, kDeal> items(a);
    while (items.next()) {
    const int rt = items.rt, bkv = items.bkv, t0 = items.t0, t1 = items.t1;
    const int b = bkv / a.kv_heads, h = (bkv % a.kv_heads) * G + items.g;
    const float* Q = reinterpret_cast<const float*>(a.q) + ((size_t)(b * a.q_heads + h) * N) * D;
    const float* K = reinterpret_cast<const float*>(a.k) + ((size_t)bkv * N) * D;
    const int lane = opaque_lane(threadIdx.x);
    const int col = lane & 31, half = lane >> 5;
    const int q_base = rt * kRows;

    unsigned dma_off[E::kOffs], frag_off[E::kKeys];
    E::dma_offsets(lane, dma_off);
    E::frag_offsets(lane, frag_off);
    const unsigned lds_k0 = lds_address(&lds_k[0][0]);

    float m_run[kSub], l_sum[kSub];                                     // running maximum, the sum relative to it
#pragma unroll
    for (int s = 0; s < kSub; ++s) { m_run[s] = -INFINITY; l_sum[s] = 0.f; }

    // Stages [from, t1), as in the second pass.
    auto sweep = [&](auto exact_c, const auto& bq, int from) __attribute__((always_inline)) {
        constexpr bool kExact = decltype(exact_c)::value;
        auto issue = [&](int t, int slot) __attribute__((always_inline)) {
            E::issue(reinterpret_cast<const char*>(K), t * kStreamRows, N, lds_k0 + slot * E::kStageBytes, dma_off);
        };
        // the reference in use (0 while nothing is seen), the sums since the last fold; what a set of stages began with
        float m_use[kSub], l_run[kSub][2], m_in[kSub], l_in[kSub];
        f32x16_t acc[2][kSub];
#pragma unroll
        for (int s = 0; s < kSub; ++s) {
            m_use[s] = 0.f; l_run[s][0] = l_run[s][1] = 0.f; m_in[s] = m_run[s]; l_in[s] = l_sum[s];
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[1][s][r] = -INFINITY;      // before the first stage: nothing seen
        }
        auto raise = [&](int s, const f32x16_t& x) __attribute__((always_inline)) {
            const float m_new = fmaxf(m_run[s], max16(x) * c);
            m_use[s] = m_new == -INFINITY ? 0.f : m_new;
            const float down = exp2_fast(m_run[s] - m_use[s]);
            l_run[s][0] *= down; l_run[s][1] *= down; l_sum[s] *= down;
            m_run[s] = m_new;
        };
        auto add = [&](int s, int r, const f32x16_t& x) __attribute__((always_inline)) {
            l_run[s][r & 1] += exp2_fast(__builtin_fmaf(x[r], c, -m_use[s]));
        };
        typename E::Feed feed;
        frag_t first = zero_frag();
        wait_lds_all_visible();
        issue(from, 0);
        wait_vmem<0>();
        if constexpr (kExact) first = E::fetch(lds_k[0], frag_off, 0);
        else feed.start(lds_k[0], frag_off);

        auto stage = [&](auto set_c, int t) __attribute__((always_inline)) {
            constexpr int set = decltype(set_c)::value;
            auto next = [&]() __attribute__((always_inline)) { wait_lds_all_visible(); if (t + 1 < t1) issue(t + 1, 1 - set); };     // (the other slot's last reads)
            auto landed = []() __attribute__((always_inline)) { wait_vmem<0>(); };
            if constexpr (!kExact) next();
            auto begin = [&](int s) __attribute__((always_inline)) { raise(s, acc[1 - set][s]); };
            auto weigh = [&](int e) __attribute__((always_inline)) { add(e & 1, e >> 1, acc[1 - set][e & 1]); };
            if constexpr (kExact) {
                E::exact_stage(lds_k[set], lds_k[1 - set], frag_off, first, bq, acc[set], next, landed, begin, weigh);
            } else {
                E::stage(lds_k[set], lds_k[1 - set], frag_off, feed, bq, acc[set], landed, begin, weigh);
            }
#pragma unroll
            for (int s = 0; s < kSub; ++s) { stays_here(l_run[s][0]); stays_here(l_run[s][1]); }
            if (t * kStreamRows + kStreamRows > q_base) {               // on the diagonal: keys after the row
                const int lane = lane_here(), col = lane & 31, half = lane >> 5;  // (nothing is kept for this)
#pragma unroll
                for (int s = 0; s < kSub; ++s)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (t * kStreamRows + acc_row(r, half) > q_base + s * 32 + col) acc[set][s][r] = -INFINITY;
            }
        };
        auto fold = [&]() __attribute__((always_inline)) {
            bool left = false;
#pragma unroll
            for (int s = 0; s < kSub; ++s) {
                l_sum[s] += l_run[s][0] + l_run[s][1];
                l_run[s][0] = l_run[s][1] = 0.f;
                left |= l_in[s] < INFINITY && !(l_sum[s] < INFINITY);
            }
            if constexpr (kExact) return false;
            const bool any = __any(left);                               // wave-uniform
#pragma unroll
            for (int s = 0; s < kSub; ++s) {
                if (any) { m_run[s] = m_in[s]; l_sum[s] = l_in[s]; }
                else { m_in[s] = m_run[s]; l_in[s] = l_sum[s]; }
            }
            return any;
        };
        int run = 2, until_fold = run;
        int t = from;
        do {
            stage(ic<0>{}, t);
            if (t + 1 < t1) stage(ic<1>{}, t + 1);
            until_fold -= 2;
            if (until_fold <= 0 && t + 2 < t1) {
                until_fold = run = min(2 * run, kFoldStagesF32);
                if (fold()) return from;
                from = t + 1;
            }
        } while ((t += 2) < t1);
        wait_vmem<0>();
        auto last = [&](const f32x16_t (&x)[kSub]) __attribute__((always_inline)) {
#pragma unroll
            for (int s = 0; s < kSub; ++s) {
                raise(s, x[s]);
#pragma unroll
                for (int r = 0; r < 16; ++r) add(s, r, x[s]);
            }
        };
        if ((t - t1) & 1) last(acc[0]);
        else last(acc[1]);
        return fold() ? from : t1;
    };
    if (t0 < t1) {                                                      // (else: a part that is padding)
        int from = t0;
        {
            Pieces bq[kSub][E::kSteps];
            const bool whole = !__any(E::load_stationary(Q, q_base, N, lane, bq));
            wait_vmem_all_visible();
            if (whole) from = scalar(sweep(std::false_type{}, bq, t0));
        }
        if (from < t1) {
            frag_t bq[kSub][E::kFrags];
            E::load_exact(Q, q_base, N, lane, bq);
            wait_vmem_all_visible();
            sweep(std::true_type{}, bq, from);
        }
    }

    const size_t bh = (size_t)(b * a.q_heads + h);
    float* lse2 = a.lse2 + bh * a.n_pad;
#pragma unroll
    for (int s = 0; s < kSub; ++s) {
        const float m_o = __shfl_xor(m_run[s], 32), l_o = __shfl_xor(l_sum[s], 32);
        const float M = fmaxf(m_run[s], m_o), Mu = M == -INFINITY ? 0.f : M;
        const float sum = l_sum[s] * exp2_fast(m_run[s] - Mu) + l_o * exp2_fast(m_o - Mu);
        const int qi = q_base + s * 32 + col;
        if constexpr (kDeal) {                                          // a part, for lse_combine_kernel
            const size_t at = (bh * (a.p1_waves + items.deal.n_units) + items.place.wave + rt) * kRows + s * 32 + col;
            if (half == 0) { a.part_m[at] = M; a.part_l[at] = sum; }
        } else {
            const float v = Mu + log2_fast(sum);
            if (half == 0 && qi < a.n_pad) lse2[qi] = qi < N ? v : INFINITY;      // rows past the end: weight zero in the second pass
            if (half == 0 && qi < N && a.lse_opt) a.lse_opt[bh * N + qi] = v * 0.693147180559945309f;
        }
    }
    }   // next work item
}

template <int D>
static void start_pass1_d(const ScoreArgs& a, bool deal, unsigned grid, hipStream_t st)
{
    if (deal) hipLaunchKernelGGL((score_pass1_f32_kernel<D, true>), dim3(grid), dim3(kWave), 0, st, a);
    else hipLaunchKernelGGL((score_pass1_f32_kernel<D, false>), dim3(grid), dim3(kWave), 0, st, a);
}
template <int D>
static void start_pass2_d(const ScoreArgs& a, bool deal, unsigned grid, hipStream_t st)
{
    if (deal) hipLaunchKernelGGL((score_pass2_f32_kernel<D, true>), dim3(grid), dim3(kWave), 0, st, a);
    else hipLaunchKernelGGL((score_pass2_f32_kernel<D, false>), dim3(grid), dim3(kWave), 0, st, a);
}
void start_pass1_f32(const ScoreArgs& a, bool deal, unsigned grid, hipStream_t st) { a.head_dim == 64 ? start_pass1_d<64>(a, deal, grid, st) : start_pass1_d<128>(a, deal, grid, st); }
void start_pass2_f32(const ScoreArgs& a, bool deal, unsigned grid, hipStream_t st) { a.head_dim == 64 ? start_pass2_d<64>(a, deal, grid, st) : start_pass2_d<128>(a, deal, grid, st); }

}  // namespace ems
