// Global / Local accumulated attention scores (Sec. 3.2) on gfx950 matrix cores.
//
// Two passes over the causal logits S = scale * Q K^T, neither of which stores an N x N
// matrix (App. A, "Global-Local Score Efficiency Discussion"):
//   pass 1 (query-stationary)  per row i: lse2_i = log2 sum_{j<=i} 2^(c S_ij), c = log2(e)
//   pass 2 (key-stationary)    per key j: sum over rows i >= j of 2^(c S_ij - lse2_i),
//                              once over all rows (global) and once over the last
//                              `window` rows (local), summed over the q-heads of a group.
// Both passes orient the MFMA so that the index being reduced over lives in the
// accumulator's registers and the index being kept lives in the lanes: reductions are
// in-register adds plus one exchange between the two half-waves, no atomics anywhere.
// Both passes run one wave per work item, one wave per SIMD (the whole register file holds
// the stationary operand), with a private LDS ring for the streamed operand.
#include "ems_common.h"
#include "ems_kernels.h"
#include "ems_score.h"
#include "ems_stream.h"

namespace ems {

static long long xcd_grid(long long n_groups, long long per_group)    // 8 x (items per XCD, padding included)
{
    return kXcds * ((n_groups + kXcds - 1) / kXcds) * per_group;
}

// Resident waves per XCD: one per SIMD.
constexpr int kXcdWaves = 128;

// Both passes' cursors; the first pass's start behind the items its waves begin with.
__global__ void score_queue_reset_kernel(int* queue)
{
    if (threadIdx.x < 2 * (kXcds + 1)) queue[threadIdx.x] = threadIdx.x > kXcds ? kXcdWaves : 0;
}

// The largest exponent of a tile that lies below the diagonal.
template <typename T, int D>
__device__ __forceinline__ float pass1_tile_max(const frag_t (&ak)[Tile<T, D>::kFrags], const frag_t (&bq)[Tile<T, D>::kFrags], float c)
{
    f32x16_t acc = zero_acc();
#pragma unroll
    for (int f = 0; f < Tile<T, D>::kFrags; ++f) mma<T>(acc, ak[f], bq[f]);
    return max16(acc) * c;
}

// Parts of a unit that the two small kernels below request together (one after the other they were most
// of 7.7 us at 1024 tokens).
constexpr int kPartsAhead = 8;

// Combines the partial (max, sum) pairs that the waves of an even deal left for a row tile into the
// row log-sum-exp, in stage order.
template <int kSub>
__global__ __launch_bounds__(256) void lse_combine_kernel(ScoreArgs a)
{
    constexpr int kRows = 32 * kSub;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const size_t bh = blockIdx.y;
    if (i >= a.n_pad) return;
    float v = INFINITY;                                           // rows past the end: weight zero in pass 2
    if (i < a.seq_len) {
        const DealPass1<kSub> deal(a.seq_len);
        const int u = i / kRows;
        const int first = deal.first(u) / a.p1_len, last = (deal.end(u) - 1) / a.p1_len;
        const size_t at = (bh * (a.p1_waves + deal.n_units) + u) * kRows + i % kRows;     // + wave * kRows
        float M = -INFINITY, L = 0.f;
        for (int w0 = first; w0 <= last; w0 += kPartsAhead) {
            float m[kPartsAhead], l[kPartsAhead];
#pragma unroll
            for (int k = 0; k < kPartsAhead; ++k) {
                const bool on = w0 + k <= last;
                m[k] = on ? a.part_m[at + (size_t)(w0 + k) * kRows] : -INFINITY;
                l[k] = on ? a.part_l[at + (size_t)(w0 + k) * kRows] : 0.f;
            }
            float top = M;
#pragma unroll
            for (int k = 0; k < kPartsAhead; ++k) top = fmaxf(top, m[k]);
            if (M > -INFINITY) L *= exp2_fast(M - top);
#pragma unroll
            for (int k = 0; k < kPartsAhead; ++k)
                if (m[k] > -INFINITY) L += l[k] * exp2_fast(m[k] - top);
            M = top;
        }
        v = M + log2_fast(L);
        if (a.lse_opt) a.lse_opt[bh * a.seq_len + i] = v * 0.693147180559945309f;
    }
    a.lse2[bh * a.n_pad + i] = v;
}

// Adds the row-chunk partial sums of pass 2 in ascending chunk order (fixed order, so the
// result does not depend on scheduling).
__global__ __launch_bounds__(256) void score_reduce_kernel(ScoreArgs a, int keys_per_block)
{
    const int N = a.seq_len;
    const int bkv = blockIdx.y;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= N) return;
    const int key_base = (j / keys_per_block) * keys_per_block;
    const int first = key_base / a.chunk_rows;       // first chunk whose rows reach this key tile
    float g = 0.f, l = 0.f;
    for (int I = first; I < a.n_chunks; ++I) {
        g += a.part_glo[((size_t)bkv * a.n_chunks + I) * N + j];
        if (I >= a.loc_chunk0)
            l += a.part_loc[((size_t)bkv * (a.n_chunks - a.loc_chunk0) + (I - a.loc_chunk0)) * N + j];
    }
    a.s_glo[(size_t)bkv * N + j] = g;
    a.s_loc[(size_t)bkv * N + j] = l;
}

// The same for an even deal: the waves that had a share of a key tile's rows, in row order.
template <int kSub>
__global__ __launch_bounds__(256) void score_reduce_deal_kernel(ScoreArgs a)
{
    constexpr int kKeys = 32 * kSub;
    const int N = a.seq_len, bkv = blockIdx.y;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= N) return;
    const DealPass2<kSub> deal(N, a.q_heads / a.kv_heads);
    const int u = j / kKeys, u0 = deal.first(u), u1 = deal.end(u);
    const int first = u0 / a.p2_len, last = (u1 - 1) / a.p2_len;
    const size_t at = ((size_t)bkv * (a.p2_waves + deal.n_units) + u) * kKeys + j % kKeys;   // + wave * kKeys
    float g = 0.f, l = 0.f;
    for (int w0 = first; w0 <= last; w0 += kPartsAhead) {
        float pg[kPartsAhead], pl[kPartsAhead];
#pragma unroll
        for (int k = 0; k < kPartsAhead; ++k) {
            const int w = w0 + k;
            const int r_begin = u * kKeys + (max(w * a.p2_len, u0) - u0) * kStreamRows;
            const int r_end = u * kKeys + (min((w + 1) * a.p2_len, u1) - u0) * kStreamRows;
            const bool on = w <= last && r_begin < N;         // (the rest is padding)
            pg[k] = on ? a.part_glo[at + (size_t)w * kKeys] : 0.f;
            pl[k] = on && r_end > N - a.window ? a.part_loc[at + (size_t)w * kKeys] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < kPartsAhead; ++k) { g += pg[k]; l += pl[k]; }
    }
    a.s_glo[(size_t)bkv * N + j] = g;
    a.s_loc[(size_t)bkv * N + j] = l;
}

// A caller's natural-log row log-sum-exp [B*Hq, N] -> the base-2, +inf-padded layout
// [B*Hq, n_pad] the second pass streams.
__global__ __launch_bounds__(256) void lse_to_base2_kernel(ScoreArgs a)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int bh = blockIdx.y;
    if (blockIdx.x == 0 && bh == 0 && threadIdx.x < 2 * (kXcds + 1)) a.queue[threadIdx.x] = 0;   // the pass that follows starts on empty queues
    if (i >= a.n_pad) return;
    a.lse2[(size_t)bh * a.n_pad + i] =
        i < a.seq_len ? a.lse_in_nat[(size_t)bh * a.seq_len + i] * 1.44269504088896340736f : INFINITY;
}


// ------------------------------------------------------------------------------------
// Pass 2, wave-private form.  A work item is ONE wave: it keeps 32 * kSub keys of one
// kv-head in registers (MFMA B operand, keys -> lanes) for its whole life and streams the
// query rows of one row chunk, 32 at a time, through an LDS ring that only this wave
// touches (DMA by this wave, read by this wave): no workgroup barrier anywhere.  One wave
// per SIMD owns the whole register file, so the stationary tile is large and every staged
// row is used for kSub MFMA tiles.
//
// The rows of a chunk fall in two classes, handled by two loops that share the ring:
//   edge rows      stages that touch the diagonal of this wave's keys or the last window:
//                  tiles are masked, skipped when above the diagonal, and (window rows) also
//                  added to the local score; a plain loop, one tile at a time;
//   interior rows  every row sees every key and no row is in the window: one software
//                  pipeline across tiles and stages.  Tiles go in pairs: the MFMA chains of
//                  the two tiles of a pair alternate (so consecutive matrix instructions never
//                  depend on each other) and between them the vector ALU turns the two
//                  accumulators the previous pair left behind into weights; the next stage's
//                  row operand and log-sum-exp are fetched from LDS into a second register set.
// 32-wide subtiles of the stationary operand per wave (8 x 8 fragments = the 256 accumulation
// registers in the 16-bit types) and LDS stages in the wave's ring
constexpr int kSub = kSubBf16, kRing = 4;
using T = bf16_t;

template <int D, bool kDeal>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(1, 1))) void score_pass2_stream_kernel(ScoreArgs a)
{
    constexpr int kFrags = Tile<T, D>::kFrags;
    constexpr int kEps = 16 / kFrags;                       // accumulator elements handled per MFMA slot
    static_assert(kFrags >= 2 && kFrags <= 16 && 16 % kFrags == 0, "slot schedule needs 2..16 fragments per row");
    constexpr int kPairs = kSub / 2;
    constexpr int kRowBytes = Tile<T, D>::kRowBytes;
    constexpr int kCpr = Tile<T, D>::kChunksPerRow;
    constexpr int kStageBytes = kStreamRows * kRowBytes;
    constexpr int kQInstr = kStageBytes / 1024;             // 16-byte DMA instructions per stage
    static_assert(kQInstr == 4 || kQInstr == 8, "one or two groups of four");
    constexpr int kLoads = kQInstr + 1;                     // + one 4-byte DMA for the rows' log-sum-exp
    static_assert((kRing - 1) * kLoads < 64, "vmcnt is a 6-bit counter");
    constexpr int kKeys = 32 * kSub;
    // stages per trip of the interior loop: after that many both the two operand register sets and
    // the ring slots are back where they started, so every slot is a compile-time constant
    constexpr int kUnroll = kRing;

    __shared__ __attribute__((aligned(1024))) char lds_q[kRing][kStageBytes];
    __shared__ __attribute__((aligned(256))) float lds_lse[kRing][2 * kStreamRows];   // second half: spare
    __shared__ float lds_sum[kDeal ? kSub : 1][kWave];      // the column sums that were set aside, a lane's own

    const float c = a.scale_log2e;
    const int N = a.seq_len, W = a.window;
    const int G = a.q_heads / a.kv_heads;

    Pass2Items<kSub, kDeal> items(a);
    while (items.next()) {
    const int bkv = items.bkv, r_begin = items.r_begin, r_end = items.r_end;
    const int key_base = items.J * kKeys;
    // [r_begin, e_end) touches the diagonal, [e_end, i_end) is interior, [i_end, r_end) holds
    // window rows (each range may be empty; all bounds but r_end are multiples of 32)
    const int win0 = N - W;
    int e_end = min(max(r_begin, min(key_base + kKeys, (win0 / kStreamRows) * kStreamRows)), r_end);
    const int i_end = min(max(e_end, (win0 / kStreamRows) * kStreamRows), r_end);
    // the interior loop takes kUnroll stages per trip: until their number divides, one more row
    // tile of every q-head goes to the edge loop (which is correct for any row)
    while ((((i_end - e_end) / kStreamRows) * G) % kUnroll) e_end += kStreamRows;

    const int b = bkv / a.kv_heads, kvh = bkv % a.kv_heads;
    const T* K = reinterpret_cast<const T*>(a.k) + ((size_t)bkv * N) * D;
    const T* Q0 = reinterpret_cast<const T*>(a.q) + ((size_t)(b * a.q_heads + kvh * G) * N) * D;
    const float* L0 = a.lse2 + (size_t)(b * a.q_heads + kvh * G) * a.n_pad;

    const int lane = opaque_lane(threadIdx.x);              // (what follows from it is formed for every item, not kept from one to the next)
    const int col = lane & 31, half = lane >> 5;

    frag_t bk[kSub][kFrags];
#pragma unroll
    for (int s = 0; s < kSub; ++s) {
        const int kj = key_base + s * 32 + col;
#pragma unroll
        for (int f = 0; f < kFrags; ++f)
            bk[s][f] = load_frag_or_zero(K, (size_t)kj * kRowBytes + f * 32 + half * 16, kj < N);
    }
    // The stationary operand lives in the accumulation registers, which only the matrix
    // instructions read: the ordinary vector registers stay free for what the ALU touches.
#pragma unroll
    for (int s = 0; s < kSub; ++s)
#pragma unroll
        for (int f = 0; f < kFrags; ++f) asm volatile("" : "+a"(bk[s][f]));

    // per-lane constants: DMA source offsets inside a stage, less what the instruction itself adds (1 KiB x its place in a
    // group of four), and the LDS offsets of this lane's operand fragments
    unsigned dma_rel[kQInstr];
#pragma unroll
    for (int j = 0; j < kQInstr; ++j) {
        const int slot = j * kWave + lane, row = slot / kCpr;
        dma_rel[j] = (unsigned)row * kRowBytes + (unsigned)(((slot % kCpr) ^ swz_key<T, D>(row)) << 4) - (unsigned)(j % 4) * 1024u;
    }
    unsigned frag_off[kFrags];
#pragma unroll
    for (int f = 0; f < kFrags; ++f)
        frag_off[f] = (unsigned)col * kRowBytes + (unsigned)(((f * 2 + half) ^ swz_key<T, D>(col)) << 4);

    const unsigned lds_q0 = lds_address(&lds_q[0][0]);
    const unsigned lds_l0 = lds_address(&lds_lse[0][0]);

    // DMA of the 32 rows starting at `row` of q-head g of the group into ring slot `slot`
    auto issue = [&](int g, int row, int slot) __attribute__((always_inline)) {
        const char* qg = reinterpret_cast<const char*>(Q0) + (size_t)g * N * kRowBytes;
        const unsigned dst = lds_q0 + slot * kStageBytes;
        if (row + kStreamRows <= N) {
            const char* base = qg + (size_t)row * kRowBytes;
#pragma unroll
            for (int j = 0; j < kQInstr; j += 4)
                dma_to_lds_x4(base, dma_rel[j], dma_rel[j + 1], dma_rel[j + 2], dma_rel[j + 3], dst + j * 1024);
        } else {                                            // rows past the end re-read the last row
#pragma unroll
            for (int j = 0; j < kQInstr; ++j) {
                const int r = (j * kWave + lane) / kCpr;
                const int over = max(row + r - (N - 1), 0);
                const unsigned off = dma_rel[j] + (unsigned)(j % 4) * 1024u;
                dma_to_lds<16>(qg, (unsigned)row * kRowBytes + off - (unsigned)over * kRowBytes, dst + j * 1024);
            }
        }
        // the rows' log-sum-exp (padded with +inf up to n_pad); both half-waves fetch the same 32
        // values, the upper half into the spare half of the slot, so that no lane is masked off
        dma_to_lds<4>(L0 + (size_t)g * a.n_pad, (unsigned)(row + col) * 4u, lds_l0 + slot * (2 * kStreamRows * 4));
    };
    // with stages issued up to `last`, wait until stage t has landed (stages complete in order)
    auto wait_landed = [&](int t, int last) __attribute__((always_inline)) {
        const int later = last - t;
        if (later >= 2) wait_vmem<2 * kLoads>();
        else if (later >= 1) wait_vmem<kLoads>();
        else wait_vmem<0>();
    };
    // LDS -> registers: this lane's operand fragments of a staged row tile, and the 16 values of
    // the rows' log-sum-exp its accumulator registers stand for
    auto fetch_frags = [&](int slot, frag_t (&q_out)[kFrags]) __attribute__((always_inline)) {
        const char* qs = lds_q[slot];
#pragma unroll
        for (int f = 0; f < kFrags; ++f) q_out[f] = *reinterpret_cast<const frag_t*>(qs + frag_off[f]);
    };
    auto fetch_lse = [&](int slot, f32x16_t& l_out) __attribute__((always_inline)) {
        const float* ls = lds_lse[slot];
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const f32x4_t v = *reinterpret_cast<const f32x4_t*>(ls + 8 * q4 + 4 * half);
#pragma unroll
            for (int i = 0; i < 4; ++i) l_out[4 * q4 + i] = v[i];
        }
    };
    auto fetch_rows = [&](int slot, frag_t (&q_out)[kFrags], f32x16_t& l_out) __attribute__((always_inline)) {
        fetch_frags(slot, q_out);
        fetch_lse(slot, l_out);
    };

    float part[kSub][kEps];
#pragma unroll
    for (int s = 0; s < kSub; ++s) {
        if constexpr (kDeal) lds_sum[s][lane] = 0.f;
#pragma unroll
        for (int e = 0; e < kEps; ++e) part[s][e] = 0.f;
    }

    wait_vmem_all_visible();

    // the vector ALU's share of one MFMA slot: kEps accumulator elements turned into weights and
    // added to the column sums, written operation by operation so that no instruction follows
    // the one it depends on (the scheduler keeps this order where it does not interleave itself)
    auto weigh = [&](float (&sum)[kEps], const f32x16_t& s_acc, const f32x16_t& l, int f) __attribute__((always_inline)) {
        float x[kEps];
#pragma unroll
        for (int e = 0; e < kEps; ++e) x[e] = __builtin_fmaf(s_acc[f * kEps + e], c, -l[f * kEps + e]);
#pragma unroll
        for (int e = 0; e < kEps; ++e) x[e] = exp2_fast(x[e]);
#pragma unroll
        for (int e = 0; e < kEps; ++e) sum[e] += x[e];
    };

    // ---- edge rows: [r_begin, e_end) and [i_end, r_end) of every q-head of the group.  A stage has
    // n_tiles key subtiles at or below the diagonal, the last of them masked when the stage is on
    // it; the chain of the next tile runs under the weights of the present one.
    float loc[kSub];
#pragma unroll
    for (int s = 0; s < kSub; ++s) loc[s] = 0.f;
    {
        const int lead = (e_end - r_begin) / kStreamRows;
        const int per_head = lead + (r_end - i_end + kStreamRows - 1) / kStreamRows;
        const int n_stages = per_head * G;
        auto row_of = [&](int u) __attribute__((always_inline)) {
            return u < lead ? r_begin + u * kStreamRows : i_end + (u - lead) * kStreamRows;
        };
        int g_next = 0, u_next = 0, u_now = 0;              // next stage to fetch (q-head, place in the head); place of the present one
        auto issue_edge = [&](int slot) __attribute__((always_inline)) {
            issue(g_next, row_of(u_next), slot);
            if (++u_next == per_head) { u_next = 0; ++g_next; }
        };
        for (int t = 0; t < kRing - 1 && t < n_stages; ++t) issue_edge(t);
        for (int t = 0; t < n_stages; ++t) {
            if (t + kRing - 1 < n_stages) issue_edge((t + kRing - 1) % kRing);
            wait_landed(t, min(n_stages - 1, t + kRing - 1));
            frag_t aq[kFrags];
            f32x16_t lse_v;
            fetch_rows(t % kRing, aq, lse_v);
            const int row0 = row_of(u_now);
            if (++u_now == per_head) u_now = 0;
            const int below = (row0 - key_base) / kStreamRows + 1;   // key subtiles at or below the diagonal
            if (row0 < win0 && row0 + 31 >= win0) {
                // the window begins inside the stage: rows are told apart element by element
#pragma unroll
                for (int ks = 0; ks < kSub; ++ks) {
                    const int ks0 = key_base + ks * 32;
                    if (ks < below)                          // wave-uniform
                        stream_edge_tile<T, D>(aq, bk[ks], lse_v, c, part[ks][0], loc[ks], row0, ks0 + col, half, win0);
                    __builtin_amdgcn_sched_barrier(0);       // one tile's temporaries at a time
                }
            } else {
                const int n_tiles = min(below, kSub);
                const int first_row = below <= kSub ? col : 0;       // the last tile's rows before it are above the diagonal
                const bool window = row0 >= win0;
                f32x16_t acc[2];
                defined_here(acc[1]);
                mma_first<T>(acc[0], aq[0], bk[0][0]);
#pragma unroll
                for (int f = 1; f < kFrags; ++f) mma<T>(acc[0], aq[f], bk[0][f]);
#pragma unroll
                for (int ks = 0; ks < kSub; ++ks) {
                    float sum[kEps];
#pragma unroll
                    for (int e = 0; e < kEps; ++e) sum[e] = 0.f;
                    const bool last = ks + 1 >= n_tiles;     // wave-uniform
                    if (ks + 1 < kSub && !last) {
                        const int kn = ks + 1 < kSub ? ks + 1 : ks;
#pragma unroll
                        for (int f = 0; f < kFrags; ++f) {
                            if (f == 0) mma_first<T>(acc[kn & 1], aq[0], bk[kn][0]);
                            else mma<T>(acc[kn & 1], aq[f], bk[kn][f]);
                            weigh(sum, acc[ks & 1], lse_v, f);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    } else {
                        float x[16];
#pragma unroll
                        for (int r = 0; r < 16; ++r) x[r] = exp2_fast(__builtin_fmaf(acc[ks & 1][r], c, -lse_v[r]));
#pragma unroll
                        for (int r = 0; r < 16; ++r) sum[r % kEps] += acc_row(r, half) < first_row ? 0.f : x[r];
                    }
#pragma unroll
                    for (int e = 0; e < kEps; ++e) part[ks][e] += sum[e];
                    if (window) {                            // wave-uniform
                        float t16 = sum[0];
#pragma unroll
                        for (int e = 1; e < kEps; ++e) t16 += sum[e];
                        loc[ks] += t16;
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if (last) break;
                }
            }
            // the slot is re-filled by the DMA issued at the top of the next iteration: the
            // fragments above are in registers by then (their uses wait for them)
        }
        wait_vmem<0>();
    }

    // ---- interior rows: [e_end, i_end) of every q-head, one pipeline over all tiles.  The loop
    // body is straight-line code (an even number of stages, DMA issued for every stage index --
    // past the end the last stage is fetched again into a ring slot nobody reads -- and a constant
    // wait count), so nothing in it can be moved out of the slot it was written in.
    if (e_end < i_end) {
        const int per_head = (i_end - e_end) / kStreamRows;
        const int n_stages = per_head * G;                  // a multiple of kUnroll

        frag_t aq[2][kFrags];
        f32x16_t lse_v[2];
        f32x16_t acc[4];
        // issue cursor of the next stage to fetch: countdowns of the stages it has left in its q-head
        // and in all.  Four DMA instructions go under one M0; the position is kept as running
        // addresses (source rows, their log-sum-exp) that advance by a stage, at the last stage of
        // a q-head by the jump to the next head's first interior row, and not at all once the last
        // stage is issued -- masks instead of selects, a dozen scalar instructions per stage.
        int h_left = per_head, t_left = n_stages;
        const char* q_src = reinterpret_cast<const char*>(Q0) + (size_t)e_end * kRowBytes;
        const char* l_src = reinterpret_cast<const char*>(L0 + e_end);
        const long long q_jump = ((long long)N - (i_end - e_end) + kStreamRows) * kRowBytes;   // last stage of a head -> next head
        const long long l_jump = ((long long)a.n_pad - (i_end - e_end) + kStreamRows) * 4;
        const unsigned lse_lane_off = (unsigned)col * 4u;
        const unsigned lds_q0s = __builtin_amdgcn_readfirstlane(lds_q0), lds_l0s = __builtin_amdgcn_readfirstlane(lds_l0);
        auto issue_next = [&](auto slot_c) __attribute__((always_inline)) {
            constexpr int slot = decltype(slot_c)::value;
            dma_to_lds_x4_at<slot * kStageBytes>(q_src, dma_rel[0], dma_rel[1], dma_rel[2], dma_rel[3], lds_q0s);
            if constexpr (kQInstr > 4)
                dma_to_lds_x4_at<slot * kStageBytes + 4096>(q_src, dma_rel[4 % kQInstr], dma_rel[5 % kQInstr],
                                                            dma_rel[6 % kQInstr], dma_rel[7 % kQInstr], lds_q0s);
            dma_dword_to_lds_at<slot * (2 * kStreamRows * 4)>(l_src, lse_lane_off, lds_l0s);
            advance_cursor<kStageBytes, kStreamRows * 4>(h_left, t_left, q_src, l_src, per_head, q_jump, l_jump);
        };

        issue_next(ic<0>{});
        issue_next(ic<1>{});
        issue_next(ic<2>{});
        wait_vmem<(kRing - 2) * kLoads>();
        fetch_rows(0, aq[0], lse_v[0]);
        // Pairs alternate between accumulators {0, 1} and {2, 3}.  The pipeline starts on a pair
        // that weighs nothing: zero logits under an infinite log-sum-exp.
#pragma unroll
        for (int r = 0; r < 16; ++r) {                      // pair 0 of stage 0 writes {0, 1} and reads {2, 3}
            acc[2][r] = acc[3][r] = 0.f;
            lse_v[1][r] = INFINITY;
        }

        // One stage = kPairs rounds.  In round p the chains of tiles 2p and 2p+1 alternate, slot by
        // slot, and after each MFMA the vector ALU weighs kEps elements of the matching tile of the
        // previous pair (for p = 0 the last pair of the previous stage, whose rows' log-sum-exp is
        // in the other register set).  An accumulator is first read two MFMAs and a dozen vector
        // instructions after the chain that wrote it has ended.
        auto stage = [&](auto u_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;         // stage t of the trip, t = u (mod kUnroll)
            constexpr int set = u & 1;
            constexpr int kFetchAt = 1;                     // as early as the other register set is free: the LDS latency has three rounds to hide in
            issue_next(ic<(u + kRing - 1) % kRing>{});      // stage t + kRing - 1
#pragma unroll
            for (int p = 0; p < kPairs; ++p) {
                const int rp = p & 1;                                          // accumulators this round writes: {2rp, 2rp+1}
                const int psa = (2 * p + kSub - 2) % kSub;                     // key subtiles of the previous pair
                f32x16_t& accA = acc[2 * rp];
                f32x16_t& accB = acc[2 * rp + 1];
                const f32x16_t& prevA = acc[2 * (1 - rp)];
                const f32x16_t& prevB = acc[2 * (1 - rp) + 1];
                const f32x16_t& pl = lse_v[p == 0 ? 1 - set : set];
#pragma unroll
                for (int f = 0; f < kFrags; ++f) {
                    if (f == 0) mma_first<T>(accA, aq[set][0], bk[2 * p][0]);
                    else mma<T>(accA, aq[set][f], bk[2 * p][f]);
                    weigh(part[psa], prevA, pl, f);
                    __builtin_amdgcn_sched_barrier(0);
                    if (f == 0) mma_first<T>(accB, aq[set][0], bk[2 * p + 1][0]);
                    else mma<T>(accB, aq[set][f], bk[2 * p + 1][f]);
                    weigh(part[psa + 1], prevB, pl, f);
                    // The other register set is free once round 0 has read the previous stage's
                    // log-sum-exp; stage t + 1 has landed once only the kRing - 2 stages issued
                    // after it are in flight.
                    if (p == kFetchAt && f == 0) {
                        wait_vmem<(kRing - 2) * kLoads>();
                        fetch_rows((u + 1) % kRing, aq[1 - set], lse_v[1 - set]);
                    }
                    // two rounds later those reads have long returned: one wait for all of them
                    if (p == kPairs - 1 && f == 0) wait_lds_all_visible();
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        const int fold = kFoldRows / kStreamRows * max(G, 2) / kUnroll * kUnroll;
        int until_fold = fold;
        for (int t = 0; t < n_stages; t += kUnroll) {
            stage(ic<0>{});
            stage(ic<1>{});
            stage(ic<2>{});
            stage(ic<3>{});
            until_fold -= kUnroll;
            if (kDeal && __builtin_expect(until_fold == 0, 0)) {     // the sums so far are set aside, in LDS (there are no registers left)
                until_fold = fold;
                const int ln = lane_here();
#pragma unroll
                for (int s = 0; s < kSub; ++s) {
                    float sum = lds_sum[s][ln];
#pragma unroll
                    for (int e = 0; e < kEps; ++e) { sum += part[s][e]; part[s][e] = 0.f; }
                    lds_sum[s][ln] = sum;
                }
            }
        }
        // the last pair (key subtiles kSub - 2 and kSub - 1 of the last stage, register set 1)
        {
            constexpr int rp = (kPairs - 1) & 1;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                part[kSub - 2][r % kEps] += exp2_fast(__builtin_fmaf(acc[2 * rp][r], c, -lse_v[1][r]));
                part[kSub - 1][r % kEps] += exp2_fast(__builtin_fmaf(acc[2 * rp + 1][r], c, -lse_v[1][r]));
            }
        }
        wait_vmem<0>();                                     // no DMA may outlive the wave's LDS
    }

    float *out_glo, *out_loc;
    items.outputs(out_glo, out_loc);
    const int out_lane = opaque_lane(lane);                 // (likewise not kept across the loops above)
#pragma unroll
    for (int s = 0; s < kSub; ++s) {
        float g = kDeal ? lds_sum[s][out_lane] : 0.f;
#pragma unroll
        for (int e = 0; e < kEps; ++e) g += part[s][e];
        const float gsum = g + __shfl(g, out_lane ^ 32);    // the half-waves hold disjoint rows of the same keys
        const float lsum = loc[s] + __shfl(loc[s], out_lane ^ 32);
        const int kj = key_base + s * 32 + out_lane;
        if (out_lane < 32 && kj < N) {
            out_glo[kj] = gsum;
            if (out_loc) out_loc[kj] = lsum;
        }
    }
    }   // next work item
}

// ------------------------------------------------------------------------------------
// Pass 1, wave-private form.  A work item is ONE wave: it keeps 32 * kSub query rows of one
// q-head in registers (MFMA B operand, queries -> lanes) and streams the keys of its share of
// the causal range, 32 at a time, through its own LDS ring (A operand, keys -> accumulator
// registers): the row sum of a query is a per-lane scalar and there is no workgroup barrier.
//
//   edge stages      the key stages that touch the diagonal of this wave's queries (masked), and
//                    those before them that do not fill a trip of the interior loop: one at a
//                    time, a tile's chain under the weights of the one before, the reference
//                    exponent m of a lane its running maximum.
//   interior stages  every key is visible to every query: the software pipeline of the second
//                    pass (paired MFMA chains, weights of the previous pair in between), with
//                    the reference m held fixed (where there are no edge stages, at the maximum of the
//                    first stage): sum += exp2(c * S - m).  Any m gives the same
//                    log-sum-exp m + log2(sum) as long as the sum stays inside the float range,
//                    i.e. no later exponent exceeds m by ~100: if a sum does leave the range,
//                    the wave redoes all of its stages in the online form (running maximum and
//                    rescaled sum, tile by tile).
// ------------------------------------------------------------------------------------
template <int D, bool kDeal>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(1, 1))) void score_pass1_stream_kernel(ScoreArgs a)
{
    constexpr int kFrags = Tile<T, D>::kFrags;
    constexpr int kEps = 16 / kFrags;
    static_assert(kFrags >= 2 && kFrags <= 16 && 16 % kFrags == 0, "slot schedule needs 2..16 fragments per row");
    constexpr int kPairs = kSub / 2;
    constexpr int kRowBytes = Tile<T, D>::kRowBytes;
    constexpr int kCpr = Tile<T, D>::kChunksPerRow;
    constexpr int kStageBytes = kStreamRows * kRowBytes;
    constexpr int kLoads = kStageBytes / 1024;              // 16-byte DMA instructions per stage
    static_assert(kLoads == 4 || kLoads == 8, "one or two groups of four");
    static_assert((kRing - 1) * kLoads < 64, "vmcnt is a 6-bit counter");
    constexpr int kRows = 32 * kSub;                        // query rows per wave
    // stages per trip of the interior loop (operand register sets and ring slots back at their start)
    constexpr int kUnroll = kRing;
    constexpr int kFold = kFoldKeys / kStreamRows / kUnroll * kUnroll;

    __shared__ __attribute__((aligned(1024))) char lds_k[kRing][kStageBytes];

    const int N = a.seq_len;
    const int G = a.q_heads / a.kv_heads;
    Pass1Items<kSub, kDeal> items(a);
    while (items.next()) {
    const int rt = items.rt, bkv = items.bkv, g = items.g, t0 = items.t0, t1 = items.t1;
    const int b = bkv / a.kv_heads, kvh = bkv % a.kv_heads;
    const int h = kvh * G + g;

    const T* Q = reinterpret_cast<const T*>(a.q) + ((size_t)(b * a.q_heads + h) * N) * D;
    const T* K = reinterpret_cast<const T*>(a.k) + ((size_t)bkv * N) * D;

    const int lane = threadIdx.x;
    const int col = lane & 31, half = lane >> 5;
    const int q_base = rt * kRows;
    const float c = a.scale_log2e;

    frag_t bq[kSub][kFrags];
#pragma unroll
    for (int s = 0; s < kSub; ++s) {
        const int qi = q_base + s * 32 + col;
#pragma unroll
        for (int f = 0; f < kFrags; ++f)
            bq[s][f] = load_frag_or_zero(Q, (size_t)qi * kRowBytes + f * 32 + half * 16, qi < N);
    }
    // the stationary operand lives in the accumulation registers (only the matrix instructions read it)
#pragma unroll
    for (int s = 0; s < kSub; ++s)
#pragma unroll
        for (int f = 0; f < kFrags; ++f) asm volatile("" : "+a"(bq[s][f]));

    unsigned dma_rel[kLoads];                               // source offsets inside a stage, as in the second pass
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
        const int slot = j * kWave + lane, row = slot / kCpr;
        dma_rel[j] = (unsigned)row * kRowBytes + (unsigned)(((slot % kCpr) ^ swz_key<T, D>(row)) << 4) - (unsigned)(j % 4) * 1024u;
    }
    unsigned frag_off[kFrags];
#pragma unroll
    for (int f = 0; f < kFrags; ++f)
        frag_off[f] = (unsigned)col * kRowBytes + (unsigned)(((f * 2 + half) ^ swz_key<T, D>(col)) << 4);
    const unsigned lds_k0 = lds_address(&lds_k[0][0]);

    // DMA of key stage t (keys 32 t ..) into ring slot `slot`
    auto issue = [&](int t, int slot) __attribute__((always_inline)) {
        const int row = t * kStreamRows;
        const unsigned dst = lds_k0 + slot * kStageBytes;
        if (row + kStreamRows <= N) {
            const char* base = reinterpret_cast<const char*>(K) + (size_t)row * kRowBytes;
#pragma unroll
            for (int j = 0; j < kLoads; j += 4)
                dma_to_lds_x4(base, dma_rel[j], dma_rel[j + 1], dma_rel[j + 2], dma_rel[j + 3], dst + j * 1024);
        } else {                                            // keys past the end re-read the last key (always masked)
#pragma unroll
            for (int j = 0; j < kLoads; ++j) {
                const int r = (j * kWave + lane) / kCpr;
                const int over = max(row + r - (N - 1), 0);
                const unsigned off = dma_rel[j] + (unsigned)(j % 4) * 1024u;
                dma_to_lds<16>(K, (unsigned)row * kRowBytes + off - (unsigned)over * kRowBytes, dst + j * 1024);
            }
        }
    };
    auto wait_landed = [&](int t, int last) __attribute__((always_inline)) {
        const int later = last - t;
        if (later >= 2) wait_vmem<2 * kLoads>();
        else if (later >= 1) wait_vmem<kLoads>();
        else wait_vmem<0>();
    };
    auto fetch_keys = [&](int slot, frag_t (&k_out)[kFrags]) __attribute__((always_inline)) {
        const char* ks = lds_k[slot];
#pragma unroll
        for (int f = 0; f < kFrags; ++f) k_out[f] = *reinterpret_cast<const frag_t*>(ks + frag_off[f]);
    };

    // of this part's key stages [t0, t1), those from t_diag on touch the diagonal
    const int t_diag = max(t0, q_base / kStreamRows);
    const int n_edge = max(t1 - t_diag, 0);
    // interior stages [t0, min(t1, t_diag)): the first n_lead of them are done in the online form, so
    // that the pipelined rest is whole trips of the loop.
    const int n_int_all = max(min(t1, t_diag) - t0, 0);
    const int n_lead = __builtin_amdgcn_readfirstlane(n_int_all % kUnroll);   // (wave-uniform; kept in a scalar register)
    const int n_int = n_int_all - n_lead;                        // a multiple of kUnroll, >= 0

    float m_run[kSub], l_run[kSub];
#pragma unroll
    for (int s = 0; s < kSub; ++s) { m_run[s] = -INFINITY; l_run[s] = 0.f; }

    // Textbook online softmax over the stages [first, end), one tile at a time.
    auto online_phase = [&](int first, int end) __attribute__((always_inline)) {
        const int n_stages = end - first;
        for (int u = 0; u < kRing - 1 && u < n_stages; ++u) issue(first + u, u % kRing);
        for (int u = 0; u < n_stages; ++u) {
            if (u + kRing - 1 < n_stages) issue(first + u + kRing - 1, (u + kRing - 1) % kRing);
            wait_landed(u, min(n_stages - 1, u + kRing - 1));
            frag_t ak[kFrags];
            fetch_keys(u % kRing, ak);
            const int key0 = (first + u) * kStreamRows;
#pragma unroll
            for (int s = 0; s < kSub; ++s) {
                const int qs0 = q_base + s * 32;
                if (key0 <= qs0 + 31)                        // wave-uniform: not entirely above the diagonal
                    pass1_tile<T, D>(ak, bq[s], m_run[s], l_run[s], c, key0, qs0 + col, half);
                __builtin_amdgcn_sched_barrier(0);           // one tile's temporaries at a time
            }
        }
        wait_vmem<0>();
    };

    // the vector ALU's share of one MFMA slot, operation by operation (no instruction follows
    // the one it depends on)
    auto weigh = [&](float (&sum)[kEps], const f32x16_t& s_acc, float m, int f) __attribute__((always_inline)) {
        float x[kEps];
#pragma unroll
        for (int e = 0; e < kEps; ++e) x[e] = __builtin_fmaf(s_acc[f * kEps + e], c, -m);
#pragma unroll
        for (int e = 0; e < kEps; ++e) x[e] = exp2_fast(x[e]);
#pragma unroll
        for (int e = 0; e < kEps; ++e) sum[e] += x[e];
    };
    float lsum[kSub][kEps];
#pragma unroll
    for (int s = 0; s < kSub; ++s)
#pragma unroll
        for (int e = 0; e < kEps; ++e) lsum[s][e] = 0.f;

    wait_vmem_all_visible();

    // ---- edge stages: the n_lead interior ones, then those on the diagonal.  Subtiles go from the
    // last one down to the one on the diagonal, which is masked; the chain of the next tile runs
    // under the weights of the present one.  The lane's reference is its running maximum: an exponent
    // far above the reference is rounded coarsely (2^-18 at 100), and its weight with it.
    const int d0 = q_base / kStreamRows;                        // subtile s is on the diagonal in stage d0 + s
    auto raise = [&](int s, const f32x16_t& x) __attribute__((always_inline)) {     // -> the reference to use (0 while nothing is seen)
        const float m_new = fmaxf(m_run[s], max16(x) * c);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        const float down = exp2_fast(m_run[s] - m_use);
#pragma unroll
        for (int e = 0; e < kEps; ++e) lsum[s][e] *= down;
        m_run[s] = m_new;
        return m_use;
    };
    {
        const int n_stages = n_lead + n_edge;
        auto stage_of = [&](int u) __attribute__((always_inline)) { return u < n_lead ? t0 + u : t_diag + (u - n_lead); };
        for (int u = 0; u < kRing - 1 && u < n_stages; ++u) issue(stage_of(u), u % kRing);
        for (int u = 0; u < n_stages; ++u) {
            if (u + kRing - 1 < n_stages) issue(stage_of(u + kRing - 1), (u + kRing - 1) % kRing);
            wait_landed(u, min(n_stages - 1, u + kRing - 1));
            frag_t ak[kFrags];
            fetch_keys(u % kRing, ak);
            const int t = stage_of(u);
            const int s_last = max(t - d0, 0);                   // the lowest subtile that sees the stage
            const int last_row = t >= d0 ? col : 31;             // its keys after this row are above the diagonal
            f32x16_t acc[2];
            defined_here(acc[kSub & 1]);
            mma_first<T>(acc[(kSub - 1) & 1], ak[0], bq[kSub - 1][0]);
#pragma unroll
            for (int f = 1; f < kFrags; ++f) mma<T>(acc[(kSub - 1) & 1], ak[f], bq[kSub - 1][f]);
#pragma unroll
            for (int s = kSub - 1; s >= 0; --s) {
                const bool last = s <= s_last;                   // wave-uniform
                if (s > 0 && !last) {
                    const int sn = s > 0 ? s - 1 : 0;
                    mma_first<T>(acc[sn & 1], ak[0], bq[sn][0]);
                    const float m = raise(s, acc[s & 1]);
#pragma unroll
                    for (int f = 0; f < kFrags; ++f) {
                        if (f > 0) mma<T>(acc[sn & 1], ak[f], bq[sn][f]);
                        weigh(lsum[s], acc[s & 1], m, f);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else {
                    f32x16_t& x = acc[s & 1];
#pragma unroll
                    for (int r = 0; r < 16; ++r) x[r] = acc_row(r, half) > last_row ? -INFINITY : x[r];
                    const float m = raise(s, x);
#pragma unroll
                    for (int f = 0; f < kFrags; ++f) weigh(lsum[s], x, m, f);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (last) break;
            }
        }
        wait_vmem<0>();
    }

    // ---- interior stages
    if (n_int > 0) {
        const int ti0 = t0 + n_lead;                             // interior stages [ti0, ti0 + n_int)

        frag_t ak[2][kFrags];
        f32x16_t acc[4];

        // issue cursor: a running source address that advances by a stage until the last stage is issued and then stays
        int t_left = n_int;
        const char* k_src = reinterpret_cast<const char*>(K) + (size_t)ti0 * kStageBytes;
        const unsigned lds_k0s = __builtin_amdgcn_readfirstlane(lds_k0);
        auto issue_next = [&](auto slot_c) __attribute__((always_inline)) {   // past the end: the last stage again, unread
            constexpr int slot = decltype(slot_c)::value;
            dma_to_lds_x4_at<slot * kStageBytes>(k_src, dma_rel[0], dma_rel[1], dma_rel[2], dma_rel[3], lds_k0s);
            if constexpr (kLoads > 4)
                dma_to_lds_x4_at<slot * kStageBytes + 4096>(k_src, dma_rel[4 % kLoads], dma_rel[5 % kLoads],
                                                            dma_rel[6 % kLoads], dma_rel[7 % kLoads], lds_k0s);
            advance_cursor<kStageBytes>(t_left, k_src);
        };
        issue_next(ic<0>{});
        issue_next(ic<1>{});
        issue_next(ic<2>{});
        wait_vmem<(kRing - 2) * kLoads>();
        fetch_keys(0, ak[0]);
        // The references stay as they are from here on: without edge stages the maxima of the first one (the
        // pipeline sums it like every other).  A lane that has seen no key yet (its half of the diagonal tile lay
        // above the diagonal) takes that of the other half, which holds the same queries.
#pragma unroll
        for (int s = 0; s < kSub; ++s) {
            if (n_edge + n_lead == 0) m_run[s] = pass1_tile_max<T, D>(ak[0], bq[s], c);      // wave-uniform
            const float m_o = __shfl_xor(m_run[s], 32);
            m_run[s] = m_run[s] == -INFINITY ? m_o : m_run[s];
            __builtin_amdgcn_sched_barrier(0);                  // one tile's temporaries at a time
        }
        // the pipeline starts on a pair that weighs nothing: exponents of -inf
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[2][r] = acc[3][r] = -INFINITY;

        // One stage = kPairs rounds; in round p the chains of query subtiles 2p and 2p+1 alternate
        // and after each MFMA the vector ALU weighs kEps elements of the matching tile of the
        // previous pair (same structure as the second pass; the exponent's offset is the lane's m).
        auto stage = [&](auto u_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;         // the stage's place in the trip
            constexpr int set = u & 1;
            issue_next(ic<(u + kRing - 1) % kRing>{});      // the stage kRing - 1 ahead
#pragma unroll
            for (int p = 0; p < kPairs; ++p) {
                const int rp = p & 1;
                const int psa = (2 * p + kSub - 2) % kSub;       // query subtiles of the previous pair
                f32x16_t& accA = acc[2 * rp];
                f32x16_t& accB = acc[2 * rp + 1];
                const f32x16_t& prevA = acc[2 * (1 - rp)];
                const f32x16_t& prevB = acc[2 * (1 - rp) + 1];
#pragma unroll
                for (int f = 0; f < kFrags; ++f) {
                    if (f == 0) mma_first<T>(accA, ak[set][0], bq[2 * p][0]);
                    else mma<T>(accA, ak[set][f], bq[2 * p][f]);
                    weigh(lsum[psa], prevA, m_run[psa], f);
                    __builtin_amdgcn_sched_barrier(0);
                    if (f == 0) mma_first<T>(accB, ak[set][0], bq[2 * p + 1][0]);
                    else mma<T>(accB, ak[set][f], bq[2 * p + 1][f]);
                    weigh(lsum[psa + 1], prevB, m_run[psa + 1], f);
                    if (p == 1 && f == 0) {   // the other register set is free; early, so that the LDS latency hides
                        wait_vmem<(kRing - 2) * kLoads>();
                        fetch_keys((u + 1) % kRing, ak[1 - set]);
                    }
                    // two rounds later those reads have long returned: one wait for all of them
                    if (p == kPairs - 1 && f == 0) wait_lds_all_visible();
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        for (int u0 = 0, run = kUnroll, fold = kUnroll; u0 < n_int;) {
            stage(ic<0>{});
            stage(ic<1>{});
            stage(ic<2>{});
            stage(ic<3>{});
            u0 += kUnroll;
            if (kDeal && __builtin_expect(u0 == fold, 0)) {
                // The sums so far are set aside, and where they have outgrown the reference their exponent goes
                // to it: after one trip, four, then every kFold stages.  (A branch in the one loop: as an
                // inner loop the stages came out 2 % slower.)
                constexpr float kHighSum = 0x1p5f;
                run = min(4 * run, kFold);
                fold += run;
                bool high = false;
#pragma unroll
                for (int s = 0; s < kSub; ++s) {
#pragma unroll
                    for (int e = 0; e < kEps; ++e) { l_run[s] += lsum[s][e]; lsum[s][e] = 0.f; }
                    high |= l_run[s] > kHighSum;
                }
                if (__any(high)) {                               // wave-uniform
#pragma unroll
                    for (int s = 0; s < kSub; ++s) give_exponent(m_run[s], l_run[s], kHighSum);
                }
            }
        }
        {   // the last pair (query subtiles kSub - 2 and kSub - 1 of the last stage, register set 1)
            constexpr int rp = (kPairs - 1) & 1;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                lsum[kSub - 2][r % kEps] += exp2_fast(__builtin_fmaf(acc[2 * rp][r], c, -m_run[kSub - 2]));
                lsum[kSub - 1][r % kEps] += exp2_fast(__builtin_fmaf(acc[2 * rp + 1][r], c, -m_run[kSub - 1]));
            }
        }
        wait_vmem<0>();

    }

    // the sums are relative to the references; one outside the float range (or NaN), or whose half-waves
    // would leave it together, sends the whole wave back through all of the part's stages in the online form
    bool bad = false;
#pragma unroll
    for (int s = 0; s < kSub; ++s) {
#pragma unroll
        for (int e = 0; e < kEps; ++e) l_run[s] += lsum[s][e];
        bad |= !(l_run[s] < 0x1p126f);
    }
    if (__any(bad)) {
#pragma unroll
        for (int s = 0; s < kSub; ++s) { m_run[s] = -INFINITY; l_run[s] = 0.f; }
        online_phase(t0, t1);
    }

    const size_t bh = (size_t)(b * a.q_heads + h);
    float* lse2 = a.lse2 + bh * a.n_pad;
    float* lse_nat = a.lse_opt ? a.lse_opt + bh * N : nullptr;
#pragma unroll
    for (int s = 0; s < kSub; ++s) {
        const float m_o = __shfl_xor(m_run[s], 32);
        const float l_o = __shfl_xor(l_run[s], 32);
        const float M = fmaxf(m_run[s], m_o);
        const float Mu = (M == -INFINITY) ? 0.f : M;
        const float L = l_run[s] * exp2_fast(m_run[s] - Mu) + l_o * exp2_fast(m_o - Mu);
        const int qi = q_base + s * 32 + col;
        if constexpr (kDeal) {
            // this part's (reference, sum); combined by lse_combine_kernel.  A sum far above its
            // reference gives its exponent to the reference: against another part's larger reference
            // 2^(M - other) could otherwise leave the float range while L still makes up for it.
            const size_t at = (bh * (a.p1_waves + items.deal.n_units) + items.place.wave + rt) * kRows + s * 32 + col;
            float m = M, l = L;
            give_exponent(m, l, 0x1p40f);
            if (half == 0) { a.part_m[at] = m; a.part_l[at] = l; }
            continue;
        }
        const float v = Mu + log2_fast(L);
        // rows past the end get +inf: the second pass then gives them weight zero
        if (half == 0 && qi < a.n_pad) lse2[qi] = qi < N ? v : INFINITY;
        if (half == 0 && qi < N && lse_nat) lse_nat[qi] = v * 0.693147180559945309f;
    }
    }   // next work item
}

int score_keys_per_block(int dtype_is_f32) { return 32 * (dtype_is_f32 ? kSubF32 : kSub); }

// How a launch's work reaches the waves; times of a pass in us, head size 128, heads x length (rows of one line were
// measured in one process, in turn).
//
// First pass, U = row tiles per resident wave.  Wide: more than one (batch, kv-head) pair per XCD, whose
// queue then holds its pairs one after the other instead of the heaviest row tiles first.
//                                                          even deal / block per item / queues
//   U < 2               deal     28 over 4, 16384    U 1.75      840 /    - /  870
//                                 8 over 2, 32768      1.0       949 /    - / 1338
//   U at 2, not wide    blocks   64 over 8, 8192       2.0       473 /  448 /  505   (a heavy and a light row tile
//                                32 over 8, 16384      2.0       913 /  876 /  908    make a pair: nothing to balance)
//                                 4 over 1, 131072     2.0      6944 / 6764 / 6786
//   2 < U < 4, not wide queues   24 over 8, 24000      2.2      1458 / 1462 / 1403
//                                28 over 4, 32768      3.5      3216 /    - / 3229
//                                 8 over 2, 98304      3.0      1.2 % in the queues' favour
//              wide     deal     4 x 32 over 8, 4096   2.0       260 /  298 /  299
//                                32 over 32, 24000     2.9      2035 /    - / 2198
//   U >= 4              queues   32 over 8, 32768      4.0      3507 /    - / 3396
//                                32 over 32, 49152     6.0      8728 /    - / 8264
//   float32 (a part's beginning is little against its stages): the deal up to U = 16
//                                 8 over 2, 16384      2.0      1283 /    - / 1267
//                                 4 x 8 over 8, 6000   2.9       753 /    - /  778
//                                32 over 8, 6000 (64)  2.9       409 /    - /  426
//                                 4 x 32 over 8, 4096  8.0      1366 /    - / 1335
//                                 4 x 32 over 32, 6000 11.8     3199 /    - / 2876
//                                 2 x 64 over 8, 8192  16.0     5019 /    - / 5032
// Second pass, by row stages per resident wave: the deal up to 1200, and always for fewer pairs than XCDs (which have
// no queues: one block per item).  Waves that stream different rows share no lines of their L2: the more rows, the
// more that costs.
//                                                    stages      deal / queues
//                                32 over 8, 8192       128       255 /  318
//                                32 over 8, 16384      512       908 /  954
//                                64 over 8, 16384     1024      1891 / 1879
//                                24 over 8, 32768     1536      2801 / 2804
//                                32 over 8, 32768     2048      3726 / 3680
//                                4 x 32 over 8, 16384 2048      4029 / 3727
//                                32 over 8, 49152     4608      8522 / 8083
//                                 6 over 2, 49152      864      1582 / 1674  (block per item)
//                                16 over 2, 65536     4096      7420 / 7419        "
//                                 4 over 1, 131072    4096      7360 / 7361        "
constexpr double kPairUnits = 1.95;        // from here to 2 a launch counts as whole pairs
constexpr double kDealStages = 1200.;
constexpr int kResident = kXcds * kXcdWaves;

template <bool kF32>
static ScoreDeal score_deal_t(int batch, int q_heads, int kv_heads, int seq_len)
{
    constexpr int kSub = kF32 ? kSubF32 : ems::kSub, kRows = 32 * kSub;
    ScoreDeal d{};
    const long long BHQ = (long long)batch * q_heads, BKV = (long long)batch * kv_heads;
    const int G = q_heads / kv_heads;
    const DealPass1<kSub> d1(seq_len);
    const double units = (double)(BHQ * d1.n_units) / 1024.;
    const bool wide = BKV > kXcds;
    bool deal1 = units < (kF32 ? 16. : wide ? 4. : 2.);
    if (!kF32 && !wide && units >= kPairUnits && units <= 2.) { d.p1_by_block = 1; deal1 = false; }
    if (deal1) {
        deal_over_waves(kResident, BHQ, d1.total(), DealPass1<kSub>::kAlign, 4, &d.p1_len, &d.p1_waves);
        d.p1_floats = (size_t)BHQ * (d.p1_waves + d1.n_units) * kRows;
    }
    const DealPass2<kSub> d2(seq_len, G);
    const double stages = 0.5 * (double)BKV * G * d2.rows_all * d2.n_units / 1024.;
    const bool fits = (d2.rows_all + 8.) * d2.n_units < 1073741824.;      // a line's stages are counted in 32 bits
    if (fits && (stages <= kDealStages || BKV < kXcds)) {
        deal_over_waves(kResident, BKV, d2.total(), DealPass2<kSub>::align(G), 1, &d.p2_len, &d.p2_waves);
        d.p2_floats = (size_t)BKV * (d.p2_waves + d2.n_units) * kRows;
    }
    return d;
}

ScoreDeal score_deal(int batch, int q_heads, int kv_heads, int seq_len, int /*head_dim*/, bool f32)
{
    return f32 ? score_deal_t<true>(batch, q_heads, kv_heads, seq_len) : score_deal_t<false>(batch, q_heads, kv_heads, seq_len);
}

// Which products: by 16x16x32 (score_m16.hip) where the launch is long enough for the chip to lower its clock, counted in stages of 32 x 256
// per resident wave, and the sequence so long that the masked stages, which cost a tenth more there, are few.  The second pass has more
// of those (its window's as well) and wins later; both passes take the same products, whose roundings of a logit then cancel (the first alone by
// 16x16x32: 16 over 16, 8191 rows, column sums weighted alike 0.9e-7 from 64 bits -> 1.1e-7).  Time by 16x16x32 over that by 32x32x16, in turn on one
// card (on another where there are two), first / second pass:
//     16 over 16, 4096   16 stages   1.00 / 1.05 (1.05)     64 over 8, 4096     64 stages    0.98 / 1.06 (1.03)
//      8 over 8, 6000    18          1.02 / 1.00            56 over 8, 4500     69           0.99 / 1.02 (1.01)
//     32 over 32, 3300   21          1.01 / 1.05 (1.08)     32 over 32, 6000    71           0.99 / 0.98 (0.97)
//      8 over 8, 8192    32          0.98 / 1.01 (0.99)     32 over 8, 6000     71           0.99 / 0.99 (0.98)
//     32 over 32, 4096   32          1.00 / 1.06 (1.01)     4 x 32 over 8, 3300 85           0.99 / 0.98
//     2 x 32 over 8, 3300 42         0.99 / 1.02 (1.01)     32 over 8, 7000     96           0.99 / 0.99
//     32 over 8, 5003    49          0.99 / 1.01 (0.98)     32 over 8, 8192    128           0.97 / 1.00
//     3 x 12 over 4, 5003 55         1.00 / 1.02 (1.02)     4 x 32 over 32, 4096 128         0.98 / 1.02
//     16 over 16, 8192   64          0.98 / 0.99 (1.00)     32 over 8, 12000   275           0.97 / 0.98
// (With the line at 16 stages, whole score calls of 3300 to 4096 rows were 2 to 3 % slower than by 32x32x16.)
// Launches of several milliseconds settle at a power limit where it depends on the chip which is faster (ms on three): 4 x 32 over 8, 16384 6.97 / 6.85,
// 7.16 / 7.23, -; 32768 28.3 / 27.5, 28.0 / 27.7, 28.0 / 29.0.  They stay with the larger products.
// With fewer (batch, kv-head) pairs than XCDs a pair's rows are streamed through several of their L2s and there is as much to lose as to win:
// 32 over 4, 32768 3416 + 3598 / 3341 + 3682, 8 over 2, 98304 8145 + 8347 / 8452 + 8227, 4 over 1, 131072 6762 + 7411 / 6684 + 7328.
constexpr double kM16Stages = 70., kM16Most = 1024.;
constexpr int kM16Rows = 3200;
static_assert(kM16Most * 1.1 < kDealStages, "a second pass by 16x16x32 products is an even deal (its stages are padded by 3 in 100 at most)");
bool score_by_16x16x32(int batch, int q_heads, int kv_heads, int seq_len, int head_dim)
{
    const DealPass1<kSub> d(seq_len);
    const double stages = 0.5 * batch * q_heads * d.n_stages * d.n_units / kResident;
    return head_dim == 128 && batch * kv_heads >= kXcds && seq_len >= kM16Rows && stages >= kM16Stages && stages <= kM16Most;
}
static bool m16_launch(const ScoreArgs& a) { return score_by_16x16x32(a.batch, a.q_heads, a.kv_heads, a.seq_len, a.head_dim); }

template <bool kF32, bool kDeal>
static void start_pass1(const ScoreArgs& a, unsigned grid, hipStream_t st)
{
    if constexpr (kF32) start_pass1_f32(a, kDeal, grid, st);
    else if (m16_launch(a)) start_pass1_m16(a, kDeal, grid, st);
    else if (a.head_dim == 64) hipLaunchKernelGGL((score_pass1_stream_kernel<64, kDeal>), dim3(grid), dim3(kWave), 0, st, a);
    else hipLaunchKernelGGL((score_pass1_stream_kernel<128, kDeal>), dim3(grid), dim3(kWave), 0, st, a);
}

template <bool kF32, bool kDeal>
static void start_pass2(const ScoreArgs& a, unsigned grid, hipStream_t st)
{
    if constexpr (kF32) start_pass2_f32(a, kDeal, grid, st);
    else if (kDeal && m16_launch(a)) start_pass2_m16(a, grid, st);
    else if (a.head_dim == 64) hipLaunchKernelGGL((score_pass2_stream_kernel<64, kDeal>), dim3(grid), dim3(kWave), 0, st, a);
    else hipLaunchKernelGGL((score_pass2_stream_kernel<128, kDeal>), dim3(grid), dim3(kWave), 0, st, a);
}

template <bool kF32>
static hipError_t launch_pass1_t(ScoreArgs& a, hipStream_t st)
{
    constexpr int kSub = kF32 ? kSubF32 : ems::kSub, kRows = 32 * kSub;
    const int BKV = a.batch * a.kv_heads, G = a.q_heads / a.kv_heads;
    const int n_row_tiles = (a.seq_len + kRows - 1) / kRows;
    ScoreArgs a1 = a;
    if (a.p1_waves) {
        const long long grid = deal_grid((long long)a.batch * a.q_heads, a.p1_waves);
        if (grid > 0x7fffffffll) return hipErrorInvalidValue;
        a.queue_clear = 0;
        start_pass1<kF32, true>(a1, (unsigned)grid, st);
        if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
        hipLaunchKernelGGL(lse_combine_kernel<kSub>, dim3((a.n_pad + 255) / 256, a.batch * a.q_heads), dim3(256), 0, st, a1);
        return hipGetLastError();
    }
    // work items of one (b, kv-head) stream the same K: one group per XCD when there are enough
    // heads to keep all XCDs busy, else groups of the G q-heads of one row tile
    if (BKV >= kXcds) { a1.p1_groups = BKV; a1.p1_per_group = n_row_tiles * G; }
    else { a1.p1_groups = BKV * n_row_tiles; a1.p1_per_group = G; }
    // one queue per XCD; resident waves.  The reset clears the second pass's cursors as well.
    const long long per_xcd = xcd_grid(a1.p1_groups, a1.p1_per_group) / kXcds;
    if (kXcds * per_xcd > 0x7fffffffll) return hipErrorInvalidValue;
    a1.p1_local = (int)per_xcd;
    a.queue_clear = !a.p1_by_block;                         // tells a second pass that follows whether its cursors are clear
    if (!a.p1_by_block) {
        hipLaunchKernelGGL(score_queue_reset_kernel, dim3(1), dim3(64), 0, st, a.queue);
        if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    }
    const unsigned grid1 = kXcds * (unsigned)(a.p1_by_block ? per_xcd : kXcdWaves);
    start_pass1<kF32, false>(a1, grid1, st);
    return hipGetLastError();
}

template <bool kF32>
static hipError_t launch_pass2_t(const ScoreArgs& a, hipStream_t st)
{
    constexpr int kSub = kF32 ? kSubF32 : ems::kSub, kKeys = 32 * kSub;
    const int BKV = a.batch * a.kv_heads;
    const int n_key_tiles = (a.seq_len + kKeys - 1) / kKeys;
    if (a.lse_in_nat) {
        dim3 g((a.n_pad + 255) / 256, a.batch * a.q_heads);
        hipLaunchKernelGGL(lse_to_base2_kernel, g, dim3(256), 0, st, a);
        if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    }
    const dim3 reduce_grid((a.seq_len + 255) / 256, BKV);
    if (a.p2_waves) {
        const long long grid = deal_grid(BKV, a.p2_waves);
        if (grid > 0x7fffffffll) return hipErrorInvalidValue;
        start_pass2<kF32, true>(a, (unsigned)grid, st);
        if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
        hipLaunchKernelGGL(score_reduce_deal_kernel<kSub>, reduce_grid, dim3(256), 0, st, a);
        return hipGetLastError();
    }
    // Queues: an XCD queue per share of the heads when they divide over the XCDs (else no queues:
    // groups dealt to the XCDs in turn, one block per pair).  The resident waves (one per SIMD:
    // 128 per XCD) draw from the cursors, and the lightest row chunks -- about 4.5 % of the items,
    // which covers the spread between XCDs; more costs more in lost L2 sharing than it balances --
    // go to the pool.
    ScoreArgs a2 = a;
    const int r_tiles = a.chunk_rows / kKeys, top = a.n_chunks - 1;
    const long long all = p2_items_upto(top, r_tiles, n_key_tiles);
    a2.q_share = BKV % kXcds == 0 ? BKV / kXcds : 0;
    a2.q_dynamic = a2.q_share != 0;
    a2.p2_split = 0;
    if (a2.q_dynamic)
        while (a2.p2_split < top && p2_items_upto(a2.p2_split, r_tiles, n_key_tiles) <= all * 45 / 1000) ++a2.p2_split;
    const long long low = p2_items_upto(a2.p2_split - 1, r_tiles, n_key_tiles);
    const long long n_local = a2.q_share * (all - low), n_pool = (long long)BKV * low;
    const long long grid2 = !a2.q_share ? xcd_grid((long long)BKV * a.n_chunks, n_key_tiles)     // no queues: a block per pair, padding included
                                        : kXcds * kXcdWaves;
    if (n_local > 0x7fffffffll || n_pool > 0x7fffffffll) return hipErrorInvalidValue;
    if (a.chunk_rows % kKeys != 0 || grid2 > 0x7fffffffll) return hipErrorInvalidValue;
    a2.p2_local = (int)n_local; a2.p2_pool = (int)n_pool;
    if (a2.q_dynamic && !a.lse_in_nat && !a.queue_clear) {  // (the conversion kernel above, or the first pass's launch, cleared them already)
        hipLaunchKernelGGL(score_queue_reset_kernel, dim3(1), dim3(64), 0, st, a.queue);
        if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    }
    start_pass2<kF32, false>(a2, (unsigned)grid2, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.n_chunks > 1) {
        hipLaunchKernelGGL(score_reduce_kernel, reduce_grid, dim3(256), 0, st, a, kKeys);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_score_pass1(ScoreArgs& a, bool f32, hipStream_t st) { return f32 ? launch_pass1_t<true>(a, st) : launch_pass1_t<false>(a, st); }
hipError_t launch_score_pass2(const ScoreArgs& a, bool f32, hipStream_t st) { return f32 ? launch_pass2_t<true>(a, st) : launch_pass2_t<false>(a, st); }

}  // namespace ems
