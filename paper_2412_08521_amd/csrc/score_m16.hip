// The two bf16 score passes at head size 128 by 16x16x32 products: what launches of about a quarter to two milliseconds run in place of score.hip's
// kernels (rule there), whose work items, partial results, ring, stages, edge and interior loops these share.
//
// A 32x32x16 product and four of 16x16x32 take the same matrix time, but these take less power, which is what limits the
// clock of a long launch, and twice the issue slots, which is what bounds a short one.  A loop of nothing but a tile's products and weights,
// without the DMA: 206 ns a tile by 32x32x16, 194 by 16x16x32.  First / second pass, us, 32x32x16 -> 16x16x32, traced in turn on one card: 32 heads over
// 8, 8000 rows 242 / 235 -> 238 / 228 (1.95 -> 2.21-2.24 GHz, matrix pipe busy 0.55 -> 0.49 of the clocks), 16384 886 / 915 -> 860 / 886 (1.80 -> 2.10 GHz,
// 0.65 -> 0.57).  (4096, which keeps the others: 77 / 80 -> 79 / 85.)  Column sums against 64 bits, 2-norm of the error over that of the sums, means of 24
// seeds, all rows (window): 4 x 32 over 8, 3300 rows 1.48e-7 -> 1.25e-7 (1.28e-7 -> 1.09e-7), 32 over 8, 8000 1.42 -> 1.37 (1.57 -> 1.42), 64 over 8, 6000 1.73 -> 1.32
// (1.64 -> 1.55), 3 x 12 over 4, 8192 1.72 -> 1.41 (2.15 -> 1.65), 8 over 8, 16384 2.22 -> 1.64 (3.10 -> 2.49), 32 over 8, 16384 8.7 -> 6.0 (16.6 -> 9.8).  With every column
// weighted alike all rows' are smaller too (0.85-2.45e-7 -> 0.67-2.39e-7), the window's between 6 % smaller and 8 % larger (64 over 8, 6000: 0.77e-7 -> 0.83e-7).
// At head size 64 the weights' exp2 are the bound and nothing is won at any length (4 x 32 over 8, 16384: 5174 / 5232).
//
// A tile is 32 rows x 32 keys, as four chains of products (two groups of 16 of the stationary rows, two halves of
// the streamed ones) that alternate, so that consecutive matrix instructions never depend on each other; the vector ALU has the weights of the tile
// before between them.
#include "ems_common.h"
#include "ems_kernels.h"
#include "ems_score.h"
#include "ems_stream.h"

namespace ems {

// 32-wide subtiles of the stationary operand per wave (16 groups of 16 x 4 fragments = the 256 accumulation
// registers) and LDS stages in the wave's ring
constexpr int kSub = kSubBf16, kRing = 4, kGroups = 2 * kSub, D = 128;
using T = bf16_t;

// A lane's share of a 32 x 32 tile: [key group][row half], register r = streamed row 16 half + 4 (lane / 16) + r of stationary row
// 16 group + lane % 16.
struct TileAcc { f32x4_t v[2][2]; };
__device__ __forceinline__ void defined_here(TileAcc& t)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("" : "=v"(t.v[i / 2][i % 2]));
}
__device__ __forceinline__ constexpr int tile_row(int h, int r, int quarter) { return 16 * h + 4 * quarter + r; }

// The streamed operand's fragments of a stage, per lane, and the products: tile `s` of the stationary operand, product i of
// 4 * kSteps in the order in which they alternate.
constexpr int kSteps = D / 32;
struct Rows { frag_t f[2][kSteps]; };
__device__ __forceinline__ void tile_product(TileAcc& t, const Rows& a, const frag_t (&b)[kGroups][kSteps], int s, int i)
{
    const int f = i / 4, k = i / 2 % 2, h = i % 2;
    t.v[k][h] = mma16(a.f[h][f], b[2 * s + k][f], f == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : t.v[k][h]);
}
__device__ __forceinline__ void tile_products(TileAcc& t, const Rows& a, const frag_t (&b)[kGroups][kSteps], int s)
{
#pragma unroll
    for (int i = 0; i < 4 * kSteps; ++i) tile_product(t, a, b, s, i);
}
// A tile in eight slots: after kSteps / 2 products the vector ALU has two elements of the tile before, those of register
// slot / 2 and key group slot % 2 in both halves.
constexpr int kSlots = 8;
__device__ __forceinline__ void slot_products(TileAcc& t, const Rows& a, const frag_t (&b)[kGroups][kSteps], int s, int slot)
{
    constexpr int kEach = 4 * kSteps / kSlots;
#pragma unroll
    for (int i = slot * kEach; i < (slot + 1) * kEach; ++i) tile_product(t, a, b, s, i);
}

// The 32 * kSub rows of X from row0 on as the stationary operand (past the end: the last row, whose results there are not
// kept; without a branch, so that all loads are in flight at once), in the accumulation registers, which only the matrix
// instructions read: the ordinary vector registers stay free for what the ALU touches.
__device__ __forceinline__ void load_stationary(const T* X, int row0, int N, int col, int quarter, frag_t (&b)[kGroups][kSteps])
{
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        const char* x = reinterpret_cast<const char*>(X) + (size_t)min(row0 + g * 16 + col, N - 1) * Tile<T, D>::kRowBytes + quarter * 16;
#pragma unroll
        for (int f = 0; f < kSteps; ++f) b[g][f] = *reinterpret_cast<const frag_t*>(x + f * 64);
    }
#pragma unroll
    for (int g = 0; g < kGroups; ++g)
#pragma unroll
        for (int f = 0; f < kSteps; ++f) asm volatile("" : "+a"(b[g][f]));
}

// LDS offsets of a lane's fragments of its row of a stage's first half (the second half's lie 16 rows on, swizzled the same way)
__device__ __forceinline__ void frag_offsets(int col, int quarter, unsigned (&off)[kSteps])
{
#pragma unroll
    for (int f = 0; f < kSteps; ++f)
        off[f] = (unsigned)col * Tile<T, D>::kRowBytes + (unsigned)(((f * 4 + quarter) ^ swz_key<T, D>(col)) << 4);
}
__device__ __forceinline__ void fetch_frags(const char* stage, const unsigned (&off)[kSteps], Rows& out)
{
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int f = 0; f < kSteps; ++f) out.f[h][f] = *reinterpret_cast<const frag_t*>(stage + h * 16 * Tile<T, D>::kRowBytes + off[f]);
}

// Source offsets of a stage's DMA for a lane, less the offset the instruction itself adds (1 KiB x its place in a group of four)
constexpr int kStageInstr = kStreamRows * Tile<T, D>::kRowBytes / 1024;
__device__ __forceinline__ void dma_offsets(int lane, unsigned (&off)[kStageInstr])
{
    static_assert(kStageInstr % 4 == 0 && kStageInstr <= 8, "one or two groups of four");
#pragma unroll
    for (int j = 0; j < kStageInstr; ++j) {
        const int slot = j * kWave + lane, row = slot / Tile<T, D>::kChunksPerRow;
        off[j] = (unsigned)row * Tile<T, D>::kRowBytes + (unsigned)(((slot % Tile<T, D>::kChunksPerRow) ^ swz_key<T, D>(row)) << 4) - (unsigned)(j % 4) * 1024u;
    }
}
// DMA of the 32 rows of X from `row` on to LDS address dst; rows past the end re-read the last row
__device__ __forceinline__ void issue_rows(const char* X, int row, int N, int lane, const unsigned (&off)[kStageInstr], unsigned dst)
{
    constexpr int kRowBytes = Tile<T, D>::kRowBytes;
    if (row + kStreamRows <= N) {
        const char* base = X + (size_t)row * kRowBytes;
#pragma unroll
        for (int j = 0; j < kStageInstr; j += 4) dma_to_lds_x4(base, off[j], off[j + 1], off[j + 2], off[j + 3], dst + j * 1024);
    } else {
#pragma unroll
        for (int j = 0; j < kStageInstr; ++j) {
            const int over = max(row + (j * kWave + lane) / Tile<T, D>::kChunksPerRow - (N - 1), 0);
            dma_to_lds<16>(X, (unsigned)row * kRowBytes + off[j] + (unsigned)(j % 4) * 1024u - (unsigned)over * kRowBytes, dst + j * 1024);
        }
    }
}
// A whole stage at a running address into ring slot `slot`
template <int slot>
__device__ __forceinline__ void issue_stage_at(const char* src, const unsigned (&off)[kStageInstr], unsigned lds0)
{
    constexpr int kStageBytes = kStreamRows * Tile<T, D>::kRowBytes, kInstr = kStageInstr;
    dma_to_lds_x4_at<slot * kStageBytes>(src, off[0], off[1], off[2], off[3], lds0);
    if constexpr (kInstr > 4)
        dma_to_lds_x4_at<slot * kStageBytes + 4096>(src, off[4 % kInstr], off[5 % kInstr], off[6 % kInstr], off[7 % kInstr], lds0);
}

// The four quarters' values of four groups of 16 stationary rows, combined: quarter q is left with group q's, i.e. a lane with that of row `lane` of
// the 64.  (Each exchange serves two groups.)
__device__ __forceinline__ void swap_halves(float& x, float& y)      // x: both lower halves, y: both upper ones
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]); y = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_rows(float& x, float& y)        // the same of neighbouring rows of 16 lanes
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]); y = __uint_as_float(r[1]);
}
__device__ __forceinline__ float groups_sum(float g0, float g1, float g2, float g3)
{
    swap_halves(g0, g2); swap_halves(g1, g3);
    float x = g0 + g2, y = g1 + g3;
    swap_rows(x, y);
    return x + y;
}
// the same of sums l relative to references m
__device__ __forceinline__ void join_sums(float& m, float& l, float m1, float l1)
{
    const float M = fmaxf(m, m1), ref = M == -INFINITY ? 0.f : M;
    l = l * exp2_fast(m - ref) + l1 * exp2_fast(m1 - ref);
    m = M;
}
__device__ __forceinline__ void groups_join(const float (&m)[kGroups], const float (&l)[kGroups], int g, float& M, float& L)
{
    float m0 = m[g], m1 = m[g + 1], m2 = m[g + 2], m3 = m[g + 3], l0 = l[g], l1 = l[g + 1], l2 = l[g + 2], l3 = l[g + 3];
    swap_halves(m0, m2); swap_halves(l0, l2); join_sums(m0, l0, m2, l2);
    swap_halves(m1, m3); swap_halves(l1, l3); join_sums(m1, l1, m3, l3);
    swap_rows(m0, m1); swap_rows(l0, l1); join_sums(m0, l0, m1, l1);
    M = m0; L = l0;
}

__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(1, 1))) void score_pass2_m16_kernel(ScoreArgs a)
{
    constexpr int kRowBytes = Tile<T, D>::kRowBytes;
    constexpr int kStageBytes = kStreamRows * kRowBytes;
    constexpr int kLoads = kStageInstr + 1;              // 16-byte DMA instructions per stage, and one of 4 bytes for the rows' log-sum-exp
    static_assert((kRing - 1) * kLoads < 64, "vmcnt is a 6-bit counter");
    constexpr int kKeys = 32 * kSub;
    // stages per trip of the interior loop: after that many both the two operand register sets and
    // the ring slots are back where they started, so every slot is a compile-time constant
    constexpr int kUnroll = kRing;

    __shared__ __attribute__((aligned(1024))) char lds_q[kRing][kStageBytes];
    __shared__ __attribute__((aligned(256))) float lds_lse[kRing][2 * kStreamRows];   // second half: spare
    __shared__ float lds_sum[kGroups][kWave];               // the column sums that were set aside, a lane's own

    const float c = a.scale_log2e;
    const int N = a.seq_len, W = a.window;
    const int G = a.q_heads / a.kv_heads;

    Pass2Items<kSub, true> items(a);
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
    const char* Q0 = reinterpret_cast<const char*>(a.q) + ((size_t)(b * a.q_heads + kvh * G) * N) * kRowBytes;
    const float* L0 = a.lse2 + (size_t)(b * a.q_heads + kvh * G) * a.n_pad;

    const int lane = opaque_lane(threadIdx.x);              // (what follows from it is formed for every item, not kept from one to the next)
    const int col = lane & 15, quarter = lane >> 4;

    frag_t bk[kGroups][kSteps];
    load_stationary(K, key_base, N, col, quarter, bk);
    unsigned dma_rel[kStageInstr], frag_off[kSteps];
    dma_offsets(lane, dma_rel);
    frag_offsets(col, quarter, frag_off);
    const unsigned lds_q0 = lds_address(&lds_q[0][0]);
    const unsigned lds_l0 = lds_address(&lds_lse[0][0]);
    // the rows' log-sum-exp (padded with +inf up to n_pad): both half-waves fetch the same 32
    // values, the upper half into the spare half of the slot, so that no lane is masked off
    const unsigned lse_lane_off = (unsigned)(lane & 31) * 4u;

    // with stages issued up to `last`, wait until stage t has landed (stages complete in order)
    auto wait_landed = [&](int t, int last) __attribute__((always_inline)) {
        const int later = last - t;
        if (later >= 2) wait_vmem<2 * kLoads>();
        else if (later >= 1) wait_vmem<kLoads>();
        else wait_vmem<0>();
    };
    // LDS -> registers: this lane's operand fragments of a staged row tile, and the values of
    // the rows' log-sum-exp its accumulator registers stand for
    struct Lse { f32x4_t v[2]; };
    auto fetch_rows = [&](int slot, Rows& q_out, Lse& l_out) __attribute__((always_inline)) {
        fetch_frags(lds_q[slot], frag_off, q_out);
#pragma unroll
        for (int h = 0; h < 2; ++h) l_out.v[h] = *reinterpret_cast<const f32x4_t*>(lds_lse[slot] + tile_row(h, 0, quarter));
    };

    float part[kGroups][2];                                 // a key's sums over the lane's rows, by row half
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        lds_sum[g][lane] = 0.f;
        part[g][0] = part[g][1] = 0.f;
    }

    wait_vmem_all_visible();

    // the vector ALU's share of a slot: two accumulator elements turned into weights and
    // added to the column sums, written operation by operation so that no instruction follows
    // the one it depends on (the scheduler keeps this order where it does not interleave itself)
    auto weigh = [&](float (&sum)[2], const TileAcc& t, const Lse& l, int slot) __attribute__((always_inline)) {
        const int k = slot % 2, r = slot / 2;
        float x[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) x[h] = __builtin_fmaf(t.v[k][h][r], c, -l.v[h][r]);
#pragma unroll
        for (int h = 0; h < 2; ++h) x[h] = exp2_fast(x[h]);
#pragma unroll
        for (int h = 0; h < 2; ++h) sum[h] += x[h];
    };

    // ---- edge rows: [r_begin, e_end) and [i_end, r_end) of every q-head of the group.  A stage has
    // n_tiles key subtiles at or below the diagonal, the last of them masked when the stage is on
    // it; the products of the next tile run under the weights of the present one.
    float loc[kGroups];
#pragma unroll
    for (int g = 0; g < kGroups; ++g) loc[g] = 0.f;
    {
        const int lead = (e_end - r_begin) / kStreamRows;
        const int per_head = lead + (r_end - i_end + kStreamRows - 1) / kStreamRows;
        const int n_stages = per_head * G;
        auto row_of = [&](int u) __attribute__((always_inline)) {
            return u < lead ? r_begin + u * kStreamRows : i_end + (u - lead) * kStreamRows;
        };
        int g_next = 0, u_next = 0, u_now = 0;              // next stage to fetch (q-head, place in the head); place of the present one
        auto issue_edge = [&](int slot) __attribute__((always_inline)) {
            const int row = row_of(u_next);
            issue_rows(Q0 + (size_t)g_next * N * kRowBytes, row, N, lane, dma_rel, lds_q0 + slot * kStageBytes);
            dma_to_lds<4>(L0 + (size_t)g_next * a.n_pad + row, lse_lane_off, lds_l0 + slot * (2 * kStreamRows * 4));
            if (++u_next == per_head) { u_next = 0; ++g_next; }
        };
        for (int t = 0; t < kRing - 1 && t < n_stages; ++t) issue_edge(t);
        for (int t = 0; t < n_stages; ++t) {
            if (t + kRing - 1 < n_stages) issue_edge((t + kRing - 1) % kRing);
            wait_landed(t, min(n_stages - 1, t + kRing - 1));
            Rows aq;
            Lse lse_v;
            fetch_rows(t % kRing, aq, lse_v);
            const int row0 = row_of(u_now);
            if (++u_now == per_head) u_now = 0;
            const int below = (row0 - key_base) / kStreamRows + 1;   // key subtiles at or below the diagonal
            if (row0 < win0 && row0 + 31 >= win0) {
                // the window begins inside the stage: rows are told apart element by element
#pragma unroll
                for (int ks = 0; ks < kSub; ++ks) {
                    if (ks < below) {                        // wave-uniform
                        TileAcc t32;
                        tile_products(t32, aq, bk, ks);
#pragma unroll
                        for (int k = 0; k < 2; ++k) {
                            const int kj = key_base + ks * 32 + k * 16 + col;
#pragma unroll
                            for (int h = 0; h < 2; ++h)
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    const int row = row0 + tile_row(h, r, quarter);
                                    const float p = row < kj ? 0.f : exp2_fast(__builtin_fmaf(t32.v[k][h][r], c, -lse_v.v[h][r]));
                                    part[2 * ks + k][h] += p;
                                    loc[2 * ks + k] += row < win0 ? 0.f : p;
                                }
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);       // one tile's temporaries at a time
                }
            } else {
                const int n_tiles = min(below, kSub);
                const bool diagonal = below <= kSub, window = row0 >= win0;      // diagonal: the last tile's rows before the key are above it
                TileAcc acc[2];
                defined_here(acc[1]);
                tile_products(acc[0], aq, bk, 0);
#pragma unroll
                for (int ks = 0; ks < kSub; ++ks) {
                    float sum[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
                    const bool last = ks + 1 >= n_tiles;     // wave-uniform
                    if (ks + 1 < kSub && !last) {
#pragma unroll
                        for (int i = 0; i < kSlots; ++i) {
                            slot_products(acc[(ks + 1) & 1], aq, bk, ks + 1 < kSub ? ks + 1 : ks, i);
                            weigh(sum[i % 2], acc[ks & 1], lse_v, i);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    } else {
#pragma unroll
                        for (int k = 0; k < 2; ++k)
#pragma unroll
                            for (int h = 0; h < 2; ++h)
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    const float x = exp2_fast(__builtin_fmaf(acc[ks & 1].v[k][h][r], c, -lse_v.v[h][r]));
                                    sum[k][h] += diagonal && tile_row(h, r, quarter) < 16 * k + col ? 0.f : x;
                                }
                    }
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        part[2 * ks + k][0] += sum[k][0];
                        part[2 * ks + k][1] += sum[k][1];
                        if (window) loc[2 * ks + k] += sum[k][0] + sum[k][1];    // wave-uniform
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

        Rows aq[2];
        Lse lse_v[2];
        TileAcc acc[2];
        // issue cursor of the next stage to fetch: countdowns of the stages it has left in its q-head
        // and in all.  Four DMA instructions go under one M0; the position is kept as running
        // addresses (source rows, their log-sum-exp) that advance by a stage, at the last stage of
        // a q-head by the jump to the next head's first interior row, and not at all once the last
        // stage is issued -- masks instead of selects, a dozen scalar instructions per stage.
        int h_left = per_head, t_left = n_stages;
        const char* q_src = Q0 + (size_t)e_end * kRowBytes;
        const char* l_src = reinterpret_cast<const char*>(L0 + e_end);
        const long long q_jump = ((long long)N - (i_end - e_end) + kStreamRows) * kRowBytes;   // last stage of a head -> next head
        const long long l_jump = ((long long)a.n_pad - (i_end - e_end) + kStreamRows) * 4;
        const unsigned lds_q0s = __builtin_amdgcn_readfirstlane(lds_q0), lds_l0s = __builtin_amdgcn_readfirstlane(lds_l0);
        auto issue_next = [&](auto slot_c) __attribute__((always_inline)) {
            constexpr int slot = decltype(slot_c)::value;
            issue_stage_at<slot>(q_src, dma_rel, lds_q0s);
            dma_dword_to_lds_at<slot * (2 * kStreamRows * 4)>(l_src, lse_lane_off, lds_l0s);
            advance_cursor<kStageBytes, kStreamRows * 4>(h_left, t_left, q_src, l_src, per_head, q_jump, l_jump);
        };

        issue_next(ic<0>{});
        issue_next(ic<1>{});
        issue_next(ic<2>{});
        wait_vmem<(kRing - 2) * kLoads>();
        fetch_rows(0, aq[0], lse_v[0]);
        // The pipeline starts on a tile that weighs nothing: zero logits under an infinite log-sum-exp.
#pragma unroll
        for (int r = 0; r < 4; ++r) {                       // tile 0 of stage 0 writes accumulators 0 and reads 1
#pragma unroll
            for (int h = 0; h < 2; ++h) { acc[1].v[0][h][r] = acc[1].v[1][h][r] = 0.f; lse_v[1].v[h][r] = INFINITY; }
        }

        // One stage = kSub tiles.  In a tile's slots the vector ALU weighs the tile before (for the first one
        // the last of the previous stage, whose rows' log-sum-exp is in the other register set).  An accumulator
        // is first read three products and a dozen vector instructions after the last that wrote it.
        auto stage = [&](auto u_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;         // stage t of the trip, t = u (mod kUnroll)
            constexpr int set = u & 1;
            constexpr int kFetchAt = 2;                     // early, once the other register set is free: the LDS latency has four tiles to hide in
            issue_next(ic<(u + kRing - 1) % kRing>{});      // stage t + kRing - 1
#pragma unroll
            for (int p = 0; p < kSub; ++p) {
                const int before = (p + kSub - 1) % kSub;
                const Lse& pl = lse_v[p == 0 ? 1 - set : set];
#pragma unroll
                for (int i = 0; i < kSlots; ++i) {
                    slot_products(acc[p & 1], aq[set], bk, p, i);
                    weigh(part[2 * before + i % 2], acc[1 - (p & 1)], pl, i);
                    // The other register set is free once tile 0 has read the previous stage's
                    // log-sum-exp; stage t + 1 has landed once only the kRing - 2 stages issued
                    // after it are in flight.
                    if (p == kFetchAt && i == 0) {
                        wait_vmem<(kRing - 2) * kLoads>();
                        fetch_rows((u + 1) % kRing, aq[1 - set], lse_v[1 - set]);
                    }
                    // four tiles later those reads have long returned: one wait for all of them
                    if (p == kFetchAt + 4 && i == 0) wait_lds_all_visible();
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
            if (__builtin_expect(until_fold == 0, 0)) {     // the sums so far are set aside, in LDS
                until_fold = fold;
                const int ln = lane_here();
#pragma unroll
                for (int g = 0; g < kGroups; ++g) {
                    lds_sum[g][ln] += part[g][0] + part[g][1];
                    part[g][0] = part[g][1] = 0.f;
                }
            }
        }
        // the last tile (accumulators 1, register set 1)
#pragma unroll
        for (int i = 0; i < kSlots; ++i) weigh(part[kGroups - 2 + i % 2], acc[1], lse_v[1], i);
        wait_vmem<0>();                                     // no DMA may outlive the wave's LDS
    }

    float *out_glo, *out_loc;
    items.outputs(out_glo, out_loc);
    const int out_lane = opaque_lane(lane);                 // (likewise not kept across the loops above)
#pragma unroll
    for (int g = 0; g < kGroups; ++g) part[g][0] = lds_sum[g][out_lane] + (part[g][0] + part[g][1]);
#pragma unroll
    for (int g = 0; g < kGroups; g += 4) {                  // the quarters hold disjoint rows of the same keys
        const int kj = key_base + g * 16 + out_lane;
        const float gv = groups_sum(part[g][0], part[g + 1][0], part[g + 2][0], part[g + 3][0]);
        const float lv = groups_sum(loc[g], loc[g + 1], loc[g + 2], loc[g + 3]);
        if (kj < N) {
            out_glo[kj] = gv;
            if (out_loc) out_loc[kj] = lv;
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
//                    time, a tile's products under the weights of the one before, the reference
//                    exponent m of a lane its running maximum.
//   interior stages  every key is visible to every query: the software pipeline of the second
//                    pass (a tile's products, weights of the previous tile in between), with
//                    the reference m held fixed (where there are no edge stages, at the maximum of the
//                    first stage): sum += exp2(c * S - m).  Any m gives the same
//                    log-sum-exp m + log2(sum) as long as the sum stays inside the float range,
//                    i.e. no later exponent exceeds m by ~100: if a sum does leave the range,
//                    the wave redoes all of its stages in the online form (running maximum and
//                    rescaled sum, tile by tile).
// ------------------------------------------------------------------------------------
template <bool kDeal>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(1, 1))) void score_pass1_m16_kernel(ScoreArgs a)
{
    constexpr int kRowBytes = Tile<T, D>::kRowBytes;
    constexpr int kStageBytes = kStreamRows * kRowBytes;
    constexpr int kLoads = kStageInstr;                  // 16-byte DMA instructions per stage
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
    const int rt = items.rt, bkv = items.bkv, g_head = items.g, t0 = items.t0, t1 = items.t1;
    const int b = bkv / a.kv_heads, kvh = bkv % a.kv_heads;
    const int h_q = kvh * G + g_head;

    const T* Q = reinterpret_cast<const T*>(a.q) + ((size_t)(b * a.q_heads + h_q) * N) * D;
    const char* K = reinterpret_cast<const char*>(a.k) + ((size_t)bkv * N) * kRowBytes;

    const int lane = opaque_lane(threadIdx.x);
    const int col = lane & 15, quarter = lane >> 4;
    const int q_base = rt * kRows;
    const float c = a.scale_log2e;

    frag_t bq[kGroups][kSteps];
    load_stationary(Q, q_base, N, col, quarter, bq);
    unsigned dma_rel[kLoads], frag_off[kSteps];
    dma_offsets(lane, dma_rel);
    frag_offsets(col, quarter, frag_off);
    const unsigned lds_k0 = lds_address(&lds_k[0][0]);

    // DMA of key stage t (keys 32 t ..) into ring slot `slot` (keys past the end re-read the last key: always masked)
    auto issue = [&](int t, int slot) __attribute__((always_inline)) {
        issue_rows(K, t * kStreamRows, N, lane, dma_rel, lds_k0 + slot * kStageBytes);
    };
    auto wait_landed = [&](int t, int last) __attribute__((always_inline)) {
        const int later = last - t;
        if (later >= 2) wait_vmem<2 * kLoads>();
        else if (later >= 1) wait_vmem<kLoads>();
        else wait_vmem<0>();
    };
    auto fetch_keys = [&](int slot, Rows& k_out) __attribute__((always_inline)) { fetch_frags(lds_k[slot], frag_off, k_out); };

    // of this part's key stages [t0, t1), those from t_diag on touch the diagonal
    const int t_diag = max(t0, q_base / kStreamRows);
    const int n_edge = max(t1 - t_diag, 0);
    // interior stages [t0, min(t1, t_diag)): the first n_lead of them are done in the online form, so
    // that the pipelined rest is whole trips of the loop.
    const int n_int_all = max(min(t1, t_diag) - t0, 0);
    const int n_lead = __builtin_amdgcn_readfirstlane(n_int_all % kUnroll);   // (wave-uniform; kept in a scalar register)
    const int n_int = n_int_all - n_lead;                        // a multiple of kUnroll, >= 0

    float m_run[kGroups], l_run[kGroups];
#pragma unroll
    for (int g = 0; g < kGroups; ++g) { m_run[g] = -INFINITY; l_run[g] = 0.f; }

    // the largest exponent of a tile's key group k
    auto tile_max = [&](const TileAcc& t, int k) __attribute__((always_inline)) {
        const f32x4_t &x = t.v[k][0], &y = t.v[k][1];
        const float t0 = fmaxf(fmaxf(x[0], x[1]), x[2]), t1 = fmaxf(fmaxf(x[3], y[0]), y[1]);
        return fmaxf(fmaxf(t0, t1), fmaxf(y[2], y[3])) * c;
    };
    // Textbook online softmax over the stages [first, end), one tile at a time.
    auto online_phase = [&](int first, int end) __attribute__((always_inline)) {
        const int n_stages = end - first;
        for (int u = 0; u < kRing - 1 && u < n_stages; ++u) issue(first + u, u % kRing);
        for (int u = 0; u < n_stages; ++u) {
            if (u + kRing - 1 < n_stages) issue(first + u + kRing - 1, (u + kRing - 1) % kRing);
            wait_landed(u, min(n_stages - 1, u + kRing - 1));
            Rows ak;
            fetch_keys(u % kRing, ak);
            const int key0 = (first + u) * kStreamRows;
#pragma unroll
            for (int s = 0; s < kSub; ++s) {
                const int qs0 = q_base + s * 32;
                if (key0 <= qs0 + 31) {                      // wave-uniform: not entirely above the diagonal
                    TileAcc t;
                    tile_products(t, ak, bq, s);
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const int g = 2 * s + k;
#pragma unroll
                        for (int h = 0; h < 2; ++h)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                if (key0 + tile_row(h, r, quarter) > qs0 + 16 * k + col) t.v[k][h][r] = -INFINITY;
                        const float m_new = fmaxf(m_run[g], tile_max(t, k));
                        const float m_use = m_new == -INFINITY ? 0.f : m_new;
                        float sum[2] = {0.f, 0.f};
#pragma unroll
                        for (int h = 0; h < 2; ++h)
#pragma unroll
                            for (int r = 0; r < 4; ++r) sum[h] += exp2_fast(__builtin_fmaf(t.v[k][h][r], c, -m_use));
                        l_run[g] = __builtin_fmaf(l_run[g], exp2_fast(m_run[g] - m_use), sum[0] + sum[1]);
                        m_run[g] = m_new;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);           // one tile's temporaries at a time
            }
        }
        wait_vmem<0>();
    };

    // the vector ALU's share of a slot, operation by operation (no instruction follows
    // the one it depends on)
    auto weigh = [&](float (&sum)[2], const TileAcc& t, float m, int slot) __attribute__((always_inline)) {
        const int k = slot % 2, r = slot / 2;
        float x[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) x[h] = __builtin_fmaf(t.v[k][h][r], c, -m);
#pragma unroll
        for (int h = 0; h < 2; ++h) x[h] = exp2_fast(x[h]);
#pragma unroll
        for (int h = 0; h < 2; ++h) sum[h] += x[h];
    };
    float lsum[kGroups][2];
#pragma unroll
    for (int g = 0; g < kGroups; ++g) lsum[g][0] = lsum[g][1] = 0.f;

    wait_vmem_all_visible();

    // ---- edge stages: the n_lead interior ones, then those on the diagonal.  Subtiles go from the
    // last one down to the one on the diagonal, which is masked; the products of the next tile run
    // under the weights of the present one.  The lane's reference is its running maximum: an exponent
    // far above the reference is rounded coarsely (2^-18 at 100), and its weight with it.
    const int d0 = q_base / kStreamRows;                        // subtile s is on the diagonal in stage d0 + s
    auto raise = [&](int s, const TileAcc& t, float (&m_use)[2]) __attribute__((always_inline)) {     // the references to use (0 while nothing is seen)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int g = 2 * s + k;
            const float m_new = fmaxf(m_run[g], tile_max(t, k));
            m_use[k] = m_new == -INFINITY ? 0.f : m_new;
            const float down = exp2_fast(m_run[g] - m_use[k]);
            lsum[g][0] *= down; lsum[g][1] *= down;
            m_run[g] = m_new;
        }
    };
    {
        const int n_stages = n_lead + n_edge;
        auto stage_of = [&](int u) __attribute__((always_inline)) { return u < n_lead ? t0 + u : t_diag + (u - n_lead); };
        for (int u = 0; u < kRing - 1 && u < n_stages; ++u) issue(stage_of(u), u % kRing);
        for (int u = 0; u < n_stages; ++u) {
            if (u + kRing - 1 < n_stages) issue(stage_of(u + kRing - 1), (u + kRing - 1) % kRing);
            wait_landed(u, min(n_stages - 1, u + kRing - 1));
            Rows ak;
            fetch_keys(u % kRing, ak);
            const int t = stage_of(u);
            const int s_last = max(t - d0, 0);                   // the lowest subtile that sees the stage
            const bool diagonal = t >= d0;                       // its keys after the query are above the diagonal
            TileAcc acc[2];
            defined_here(acc[kSub & 1]);
            tile_products(acc[(kSub - 1) & 1], ak, bq, kSub - 1);
#pragma unroll
            for (int s = kSub - 1; s >= 0; --s) {
                const bool last = s <= s_last;                   // wave-uniform
                TileAcc& x = acc[s & 1];
                float m[2];
                if (s > 0 && !last) {
                    slot_products(acc[(s - 1) & 1], ak, bq, s > 0 ? s - 1 : 0, 0);
                    raise(s, x, m);
#pragma unroll
                    for (int i = 0; i < kSlots; ++i) {
                        if (i > 0) slot_products(acc[(s - 1) & 1], ak, bq, s > 0 ? s - 1 : 0, i);
                        weigh(lsum[2 * s + i % 2], x, m[i % 2], i);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int h = 0; h < 2; ++h)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                x.v[k][h][r] = diagonal && tile_row(h, r, quarter) > 16 * k + col ? -INFINITY : x.v[k][h][r];
                    raise(s, x, m);
#pragma unroll
                    for (int i = 0; i < kSlots; ++i) weigh(lsum[2 * s + i % 2], x, m[i % 2], i);
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

        Rows ak[2];
        TileAcc acc[2];

        // issue cursor: a running source address that advances by a stage until the last stage is issued and then stays
        int t_left = n_int;
        const char* k_src = K + (size_t)ti0 * kStageBytes;
        const unsigned lds_k0s = __builtin_amdgcn_readfirstlane(lds_k0);
        auto issue_next = [&](auto slot_c) __attribute__((always_inline)) {   // past the end: the last stage again, unread
            issue_stage_at<decltype(slot_c)::value>(k_src, dma_rel, lds_k0s);
            advance_cursor<kStageBytes>(t_left, k_src);
        };
        issue_next(ic<0>{});
        issue_next(ic<1>{});
        issue_next(ic<2>{});
        wait_vmem<(kRing - 2) * kLoads>();
        fetch_keys(0, ak[0]);
        // The references stay as they are from here on: without edge stages the maxima of the first one (the
        // pipeline sums it like every other).  A lane that has seen no key yet (its quarter of the diagonal tile lay
        // above the diagonal) takes the largest of the other quarters, which hold the same queries.
#pragma unroll
        for (int s = 0; s < kSub; ++s) {
            if (n_edge + n_lead == 0) {                          // wave-uniform
                TileAcc t;
                tile_products(t, ak[0], bq, s);
#pragma unroll
                for (int k = 0; k < 2; ++k) m_run[2 * s + k] = tile_max(t, k);
            }
            __builtin_amdgcn_sched_barrier(0);                  // one tile's temporaries at a time
        }
        bool unseen = false;
#pragma unroll
        for (int g = 0; g < kGroups; ++g) unseen |= m_run[g] == -INFINITY;
        if (__any(unseen)) {                                    // wave-uniform
#pragma unroll
            for (int g = 0; g < kGroups; ++g) {
                const float top = quarters_max(m_run[g]);
                m_run[g] = m_run[g] == -INFINITY ? top : m_run[g];
            }
        }
        // the pipeline starts on a tile that weighs nothing: exponents of -inf
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[1].v[i / 2][i % 2] = f32x4_t{-INFINITY, -INFINITY, -INFINITY, -INFINITY};

        // One stage = kSub tiles; in a tile's slots the vector ALU weighs the tile before
        // (same structure as the second pass; the exponent's offset is the lane's m).
        auto stage = [&](auto u_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;         // the stage's place in the trip
            constexpr int set = u & 1, kFetchAt = 2;
            issue_next(ic<(u + kRing - 1) % kRing>{});      // the stage kRing - 1 ahead
#pragma unroll
            for (int p = 0; p < kSub; ++p) {
                const int before = (p + kSub - 1) % kSub;
#pragma unroll
                for (int i = 0; i < kSlots; ++i) {
                    slot_products(acc[p & 1], ak[set], bq, p, i);
                    weigh(lsum[2 * before + i % 2], acc[1 - (p & 1)], m_run[2 * before + i % 2], i);
                    if (p == kFetchAt && i == 0) {   // the other register set is free; early, so that the LDS latency hides
                        wait_vmem<(kRing - 2) * kLoads>();
                        fetch_keys((u + 1) % kRing, ak[1 - set]);
                    }
                    // four tiles later those reads have long returned: one wait for all of them
                    if (p == kFetchAt + 4 && i == 0) wait_lds_all_visible();
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
                for (int g = 0; g < kGroups; ++g) {
                    l_run[g] += lsum[g][0] + lsum[g][1];
                    lsum[g][0] = lsum[g][1] = 0.f;
                    high |= l_run[g] > kHighSum;
                }
                if (__any(high)) {                               // wave-uniform
#pragma unroll
                    for (int g = 0; g < kGroups; ++g) give_exponent(m_run[g], l_run[g], kHighSum);
                }
            }
        }
        // the last tile (accumulators 1, register set 1)
#pragma unroll
        for (int i = 0; i < kSlots; ++i) weigh(lsum[kGroups - 2 + i % 2], acc[1], m_run[kGroups - 2 + i % 2], i);
        wait_vmem<0>();

    }

    // the sums are relative to the references; one outside the float range (or NaN), or whose quarter-waves
    // would leave it together, sends the whole wave back through all of the part's stages in the online form
    bool bad = false;
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        l_run[g] += lsum[g][0] + lsum[g][1];
        bad |= !(l_run[g] < 0x1p125f);
    }
    if (__any(bad)) {
#pragma unroll
        for (int g = 0; g < kGroups; ++g) { m_run[g] = -INFINITY; l_run[g] = 0.f; }
        online_phase(t0, t1);
    }

    const size_t bh = (size_t)(b * a.q_heads + h_q);
    float* lse2 = a.lse2 + bh * a.n_pad;
    float* lse_nat = a.lse_opt ? a.lse_opt + bh * N : nullptr;
#pragma unroll
    for (int g = 0; g < kGroups; g += 4) {
        const int row = g * 16 + lane, qi = q_base + row;
        float m, l;
        groups_join(m_run, l_run, g, m, l);
        if constexpr (kDeal) {
            // this part's (reference, sum); combined by lse_combine_kernel.  A sum far above its
            // reference gives its exponent to the reference: against another part's larger reference
            // 2^(M - other) could otherwise leave the float range while L still makes up for it.
            const size_t at = (bh * (a.p1_waves + items.deal.n_units) + items.place.wave + rt) * kRows + row;
            give_exponent(m, l, 0x1p40f);
            a.part_m[at] = m; a.part_l[at] = l;
            continue;
        }
        const float v = (m == -INFINITY ? 0.f : m) + log2_fast(l);
        // rows past the end get +inf: the second pass then gives them weight zero
        if (qi < a.n_pad) lse2[qi] = qi < N ? v : INFINITY;
        if (qi < N && lse_nat) lse_nat[qi] = v * 0.693147180559945309f;
    }
    }   // next work item
}

void start_pass1_m16(const ScoreArgs& a, bool deal, unsigned grid, hipStream_t st)
{
    if (deal) hipLaunchKernelGGL(score_pass1_m16_kernel<true>, dim3(grid), dim3(kWave), 0, st, a);
    else hipLaunchKernelGGL(score_pass1_m16_kernel<false>, dim3(grid), dim3(kWave), 0, st, a);
}

void start_pass2_m16(const ScoreArgs& a, unsigned grid, hipStream_t st)
{
    hipLaunchKernelGGL(score_pass2_m16_kernel, dim3(grid), dim3(kWave), 0, st, a);
}

}  // namespace ems
