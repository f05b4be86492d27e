// Head-wise evict-then-merge (Sec. 4.2, Eq. 5, App. A).
//
// dest_kernel     for every to-be-merged (TBM) token: cosine similarity of its key with
//                 the class-centre keys as an MFMA contraction of the raw keys, scaled by
//                 the reciprocal norms afterwards, with the row arg-max fused into the
//                 accumulator read-out; similarity not above tau -> zero class.  With many
//                 centres the centre list is cut into slices, one block per (128 or 256
//                 tokens, slice), and dest_combine_kernel takes the best slice per token.
// merge_kernel    one to eight output rows per wave: a centre slot gathers the TBM tokens
//                 sent to it and averages (unit keys scaled by the centre's norm, raw
//                 values); one block per head, or several that leave their sums for the
//                 last of them to add in block order, do the same for the zero class; the
//                 local-window rows are copied.  Every output element has exactly one
//                 writer and every sum a fixed order; the one atomic counts the arrivals
//                 of the zero class's blocks, so results are reproducible bit for bit.
#include "ems_common.h"
#include "ems_kernels.h"
#include "ems_rows.h"

#include <algorithm>
#include <type_traits>

namespace ems {

constexpr int kMrgWaves = 4;
constexpr int kMrgBlock = kMrgWaves * kWave;
constexpr int kDestDepth = 4;        // centre stages whose rows a block has in flight at once, at most
constexpr int kDestMaxSlices = 16;   // centre slices per head at most
constexpr int kMergeWaves = 8;       // output rows per merge block
constexpr int kMergeBlock = kMergeWaves * kWave;
constexpr int kMergeStretch = 512;   // TBM tokens that a wave of a merge block sifts at a time
constexpr int kMergeMaxRows = 8;     // output rows per wave of a merge block at most
constexpr int kMergeFew = 4;         // members up to which a slot is one lane group's work
constexpr int kZeroTokens = 512;     // TBM tokens per block of a shared zero class

template <typename T> struct DestCfg { static constexpr int kStageRows = 64; };
template <> struct DestCfg<float> { static constexpr int kStageRows = 32; };

// Blocks are dealt to the 8 XCDs in turn by their index; each XCD takes consecutive (head, block of the
// head) pairs, so that the rows of a head are gathered into one L2 by every kernel of the stage (4032
// centres, 4096 tokens, 8 heads: a head's keys are 2 MB of the 4 MB, all heads' 16 MB).
constexpr int kMrgXcds = 8;
struct HeadBlock { int head, block; };
__device__ __forceinline__ HeadBlock head_block(int heads, int per_head)
{
    const int n = heads * per_head, per_xcd = (n + kMrgXcds - 1) / kMrgXcds;
    const int i = blockIdx.x / kMrgXcds, w = (int)(blockIdx.x % kMrgXcds) * per_xcd + i;
    if (i >= per_xcd || w >= n) return {-1, 0};
    return {w / per_head, w % per_head};
}
static long long head_grid(long long heads, long long per_head) { return kMrgXcds * ((heads * per_head + kMrgXcds - 1) / kMrgXcds); }

__device__ __forceinline__ int clamp_pos(int p, int n) { return min(max(p, 0), n - 1); }

// ------------------------------------------------------------------------------------
// Destination of every TBM token (Eq. 5, then the threshold).  The redundancy is the key
// cosine, the value cosine or their product (Sec. 4.1; similarity ablation of App. B):
// kSim = 0 / 1 / 2, i.e. one or two sources, each with its own MFMA contraction.
// Block = (128 * kTok TBM tokens, one slice of the centres, one (b, kv-head)); each wave keeps
// 32 * kTok TBM rows in registers as the MFMA B operand (tokens -> lanes) and the centre rows stream
// through LDS as the A operand (centres -> accumulator registers), so the running arg-max is a
// per-lane pair.  A centre row is gathered once per token tile: with many tokens larger tiles pay.
//
// What bounds it: a 32 x 32 tile is 256 clocks of products and 192 of scaling and comparing, which two waves per SIMD
// overlap; beside them a stage's norms, and at a block's beginning two dependent gathers with nothing to do meanwhile.
// So a slice is long where there are tokens enough to fill the chip (dest_cost), its gathers run a round ahead of its products
// through one barrier a stage, and its norms are one root per lane.  Destination and merge, slices of one round with the
// rows requested between barriers before, now: 8 heads, 4032 centres, 4096 tokens 83.7 -> 60 us; 96 heads, 1968, 2000
// 264 -> 194; 8 heads, 448, 512 by the product of cosines 31.3 -> 21.0, 4032, 4096 286 -> 166.
// ------------------------------------------------------------------------------------
template <typename T, int D, int kSim, int kTok>
__global__ __launch_bounds__(kMrgBlock, kSim == 2 ? 1 : 2) void dest_kernel(MergeArgs a)
{
    constexpr int kStageRows = DestCfg<T>::kStageRows;
    constexpr int kFrags = Tile<T, D>::kFrags;
    constexpr int kStride = Tile<T, D>::kLdsStride;
    constexpr int kCpr = Tile<T, D>::kChunksPerRow;
    constexpr int kPerThread = kCpr * kStageRows / kMrgBlock;
    constexpr int kSrc = kSim == 2 ? 2 : 1;
    constexpr int kDepth = kTok * kSrc * Tile<T, D>::kFrags > 8 ? 2 : kDestDepth;    // (as registers allow)

    // two stages, so that one barrier per stage is enough: whoever writes a stage has passed the barrier that
    // its other readers reached after the one before it
    __shared__ __attribute__((aligned(16))) char lds[2][kSrc][kStageRows * kStride];
    __shared__ __attribute__((aligned(16))) float lds_rn[2][kSrc][kStageRows];

    const int N = a.seq_len, n_imp = a.n_imp, n_tbm = a.n_tbm;
    const int tiles = (n_tbm + kMrgWaves * 32 * kTok - 1) / (kMrgWaves * 32 * kTok);
    const HeadBlock hb = head_block(a.bkv, tiles * a.n_slices);
    if (hb.head < 0) return;                                // block-uniform
    const int bkv = hb.head, slice = hb.block / tiles, tile = hb.block % tiles;
    const int c_begin = slice * a.slice_rows, c_end = min(n_imp, c_begin + a.slice_rows);   // this block's centres
    const T* K = reinterpret_cast<const T*>(a.k) + ((size_t)bkv * N) * D;
    const T* V = reinterpret_cast<const T*>(a.v) + ((size_t)bkv * N) * D;
    const T* src[kSrc];
    if constexpr (kSim == 0) { src[0] = K; }
    else if constexpr (kSim == 1) { src[0] = V; }
    else { src[0] = K; src[1] = V; }
    const int32_t* tbm = a.tbm_idx + (size_t)bkv * n_tbm;
    const int32_t* imp = n_imp ? a.imp_idx + (size_t)bkv * n_imp : tbm;   // (without centres the loads below still find a list)

    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int col = lane & 31, half = lane >> 5;
    const int ti0 = (tile * kMrgWaves + wave) * (32 * kTok) + col;   // this lane's first TBM token (of kTok, 32 apart)

    // A round is kDepth stages of kStageRows centres.  The first round's positions, then its rows, share their
    // round trips with the tokens'; from then on a stage's registers take its rows of the next round as soon as
    // they are in LDS, from positions that a round's work has had to arrive.
    // (Past the slice's end: its last centre, whose products a NaN of a norm takes out.  No branch here, so that the
    // loads stay in flight across the barriers.)
    int pos_pf[kDepth][kPerThread];
    frag_t pf[kDepth][kSrc][kPerThread];
    auto request_positions = [&](int st, int r0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kPerThread; ++i)
            pos_pf[st][i] = imp[min(r0 + st * kStageRows + (int)(threadIdx.x + i * kMrgBlock) / kCpr, max(c_end - 1, 0))];
    };
    auto request_rows = [&](int st) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kPerThread; ++i) {
            const int cc = (threadIdx.x + i * kMrgBlock) % kCpr;
#pragma unroll
            for (int s = 0; s < kSrc; ++s)
                pf[st][s][i] = *reinterpret_cast<const frag_t*>(reinterpret_cast<const char*>(src[s]) + ((size_t)clamp_pos(pos_pf[st][i], N) * kCpr + cc) * 16);
        }
    };

    frag_t bt[kTok][kSrc][kFrags], kt[kSim == 1 ? kTok : 1][kFrags];
    float t_rn[kTok][kSrc], k_sumsq[kTok];
    int t_pos[kTok];
#pragma unroll
    for (int tk = 0; tk < kTok; ++tk) t_pos[tk] = ti0 + 32 * tk < n_tbm ? clamp_pos(tbm[ti0 + 32 * tk], N) : 0;
#pragma unroll
    for (int st = 0; st < kDepth; ++st) request_positions(st, c_begin);
#pragma unroll
    for (int tk = 0; tk < kTok; ++tk) {                              // (a lane past the list's end: any row, its result is not kept)
#pragma unroll
        for (int s = 0; s < kSrc; ++s)
#pragma unroll
            for (int f = 0; f < kFrags; ++f)
                bt[tk][s][f] = *reinterpret_cast<const frag_t*>(reinterpret_cast<const char*>(src[s]) + (size_t)t_pos[tk] * Tile<T, D>::kRowBytes + f * 32 + half * 16);
        if constexpr (kSim == 1) {                                  // the key norm is an output in every mode
#pragma unroll
            for (int f = 0; f < kFrags; ++f)
                kt[tk][f] = *reinterpret_cast<const frag_t*>(reinterpret_cast<const char*>(K) + (size_t)t_pos[tk] * Tile<T, D>::kRowBytes + f * 32 + half * 16);
        }
    }
    constexpr int kRound = kDepth * kStageRows;
#pragma unroll
    for (int st = 0; st < kDepth; ++st) {
        request_rows(st);
        request_positions(st, c_begin + kRound);
    }
#pragma unroll
    for (int tk = 0; tk < kTok; ++tk) {
#pragma unroll
        for (int s = 0; s < kSrc; ++s) {
            float ss = 0.f;
#pragma unroll
            for (int f = 0; f < kFrags; ++f) ss += frag_sumsq<T>(bt[tk][s][f]);
            ss += __shfl_xor(ss, 32);
            t_rn[tk][s] = inv_norm(ss);
            if (s == 0) k_sumsq[tk] = ss;
        }
        if constexpr (kSim == 1) {
            float ss = 0.f;
#pragma unroll
            for (int f = 0; f < kFrags; ++f) ss += frag_sumsq<T>(kt[tk][f]);
            k_sumsq[tk] = ss + __shfl_xor(ss, 32);
        }
    }

    // A token's own norm is applied to its maximum only.  A factor of zero (a row of zeros, one whose squares
    // leave the float range, one that holds an infinity or a NaN) would lose the products' order, and times an
    // infinite maximum be no number: a wave that holds such a token applies the factors to every product.
    float best[kTok];
    int arg[kTok];
    bool no_factor = false;
#pragma unroll
    for (int tk = 0; tk < kTok; ++tk) { best[tk] = -INFINITY; arg[tk] = 0; no_factor |= t_rn[tk][0] == 0.f; }
    const bool each = kSrc == 1 && __any(no_factor);

    auto stage = [&](auto whole, int st, int c0) __attribute__((always_inline)) {
        constexpr bool kWhole = decltype(whole)::value;        // of a round that lies in the slice
        const int b = st & 1;                                  // (a round is an even number of stages)
        // the kCpr consecutive lanes that hold a row add up its squares; of the rows that they hold in turn, the
        // i-th lane does the i-th one's norm
        float ss[kSrc];
#pragma unroll
        for (int i = 0; i < kPerThread; ++i) {
            const int c = threadIdx.x + i * kMrgBlock;
            const int row = c / kCpr, cc = c % kCpr;
#pragma unroll
            for (int s = 0; s < kSrc; ++s) {
                *reinterpret_cast<frag_t*>(lds[b][s] + row * kStride + cc * 16) = pf[st][s][i];
                const float sum = group_sum<kCpr>(frag_sumsq<T>(pf[st][s][i]));
                ss[s] = i == 0 || cc == i ? sum : ss[s];
            }
        }
        {
            const int i = threadIdx.x % kCpr, row = threadIdx.x / kCpr + i * (kMrgBlock / kCpr);
            if (i < kPerThread) {
#pragma unroll
                for (int s = 0; s < kSrc; ++s) lds_rn[b][s][row] = c0 + row < c_end ? row_inv_norm<T>(ss[s]) : __builtin_nanf("");
            }
        }
        if constexpr (kWhole) {
            request_rows(st);
            request_positions(st, c0 + 2 * kRound - st * kStageRows);
        }
        __syncthreads();
#pragma unroll
        for (int rs = 0; rs < kStageRows / 32; ++rs) {
            const int cbase = c0 + rs * 32;
            if (!kWhole && cbase >= c_end) continue;       // block-uniform
            f32x16_t acc[kTok][kSrc];
#pragma unroll
            for (int s = 0; s < kSrc; ++s) {
#pragma unroll
                for (int f = 0; f < kFrags; ++f) {
                    const frag_t ac = *reinterpret_cast<const frag_t*>(lds[b][s] + (rs * 32 + col) * kStride + f * 32 + half * 16);
#pragma unroll
                    for (int tk = 0; tk < kTok; ++tk) {
                        if (f == 0) mma_first<T>(acc[tk][s], ac, bt[tk][s][f]);
                        else mma<T>(acc[tk][s], ac, bt[tk][s][f]);
                    }
                }
            }
            if (each) {                                    // wave-uniform
#pragma unroll
                for (int tk = 0; tk < kTok; ++tk)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[tk][0][r] *= t_rn[tk][0];
            }
            // Three operations per element: pairs of centres are compared with the best so far, the winning
            // pair is noted by its first register (a constant) and that one's value, the tile by one select per tile.
            float before[kTok], first[kTok];
            int reg[kTok];
#pragma unroll
            for (int tk = 0; tk < kTok; ++tk) { before[tk] = best[tk]; first[tk] = 0.f; reg[tk] = 0; }
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                f32x4_t rn[kSrc];                          // NaN past the slice's end: never the larger one
#pragma unroll
                for (int s = 0; s < kSrc; ++s)
                    rn[s] = *reinterpret_cast<const f32x4_t*>(lds_rn[b][s] + rs * 32 + 8 * q4 + 4 * half);
#pragma unroll
                for (int tk = 0; tk < kTok; ++tk)
#pragma unroll
                    for (int e = 0; e < 4; e += 2) {
                        float sim[2];
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            sim[i] = acc[tk][0][4 * q4 + e + i] * rn[0][e + i];
                            if constexpr (kSrc == 2) sim[i] = (sim[i] * t_rn[tk][0]) * ((acc[tk][1][4 * q4 + e + i] * rn[1][e + i]) * t_rn[tk][1]);
                        }
                        const float top = fmaxf(fmaxf(sim[0], sim[1]), best[tk]);      // (NaN counts as the smallest)
                        const bool won = top > best[tk];
                        reg[tk] = won ? 4 * q4 + e : reg[tk];
                        first[tk] = won ? sim[0] : first[tk];
                        best[tk] = top;
                    }
            }
#pragma unroll
            for (int tk = 0; tk < kTok; ++tk)              // (the second of the pair only where it is the larger one)
                if (best[tk] > before[tk]) arg[tk] = cbase + acc_row(reg[tk] + (first[tk] == best[tk] ? 0 : 1), half);
        }
    };
    int r0 = c_begin;
    for (; r0 + kRound <= c_end; r0 += kRound) {
#pragma unroll
        for (int st = 0; st < kDepth; ++st) stage(std::true_type{}, st, r0 + st * kStageRows);
    }
#pragma unroll
    for (int st = 0; st < kDepth; ++st)
        if (r0 + st * kStageRows < c_end) stage(std::false_type{}, st, r0 + st * kStageRows);     // block-uniform
#pragma unroll
    for (int tk = 0; tk < kTok; ++tk) {
        if constexpr (kSrc == 1)
            if (!each && best[tk] > -INFINITY) best[tk] *= t_rn[tk][0];
        // the other half-wave looked at the other centres of every tile
        const float best_o = __shfl_xor(best[tk], 32);
        const int arg_o = __shfl_xor(arg[tk], 32);
        if (best_o > best[tk] || (best_o == best[tk] && arg_o < arg[tk])) { best[tk] = best_o; arg[tk] = arg_o; }
        const int ti = ti0 + 32 * tk;
        if (half == 0 && ti < n_tbm) {
            if (a.n_slices == 1) {
                a.tbm_sim[(size_t)bkv * n_tbm + ti] = best[tk];
                a.tbm_dest[(size_t)bkv * n_tbm + ti] = best[tk] > a.tau ? arg[tk] : a.budget;
            } else {
                a.part_best[((size_t)bkv * a.n_slices + slice) * n_tbm + ti] = best[tk];
                a.part_arg[((size_t)bkv * a.n_slices + slice) * n_tbm + ti] = arg[tk];
            }
            if (slice == 0) a.k_norm[(size_t)bkv * (n_imp + n_tbm) + n_imp + ti] = sqrtf(k_sumsq[tk]);
        }
    }
}

// The best slice of every TBM token (lowest slice, hence lowest centre, on ties), then the
// threshold.  One thread per token.  Also clears the count of the zero class, on which the merge's
// blocks count their arrivals.
__global__ __launch_bounds__(kMrgBlock) void dest_combine_kernel(MergeArgs a)
{
    const int bkv = blockIdx.y, ti = blockIdx.x * kMrgBlock + threadIdx.x;
    if (ti == 0) a.slot_count[(size_t)bkv * (a.n_imp + 1) + a.n_imp] = 0;
    if (ti >= a.n_tbm) return;
    const float* pb = a.part_best + (size_t)bkv * a.n_slices * a.n_tbm + ti;
    const int32_t* pa = a.part_arg + (size_t)bkv * a.n_slices * a.n_tbm + ti;
    float b[kDestMaxSlices];
    int g[kDestMaxSlices];
#pragma unroll
    for (int s = 0; s < kDestMaxSlices; ++s) {               // every slice requested before the first compare
        const bool on = s < a.n_slices;
        b[s] = on ? pb[(size_t)s * a.n_tbm] : -INFINITY;
        g[s] = on ? pa[(size_t)s * a.n_tbm] : 0;
    }
    float best = -INFINITY;
    int arg = 0;
#pragma unroll
    for (int s = 0; s < kDestMaxSlices; ++s)
        if (b[s] > best) { best = b[s]; arg = g[s]; }
    a.tbm_sim[(size_t)bkv * a.n_tbm + ti] = best;
    a.tbm_dest[(size_t)bkv * a.n_tbm + ti] = best > a.tau ? arg : a.budget;
}

// ------------------------------------------------------------------------------------
// Segmented average.  A row of D elements is 16-byte pieces over kLpr lanes, so one wave
// has kGroups = 64 / kLpr rows in flight per load; members of a slot are dealt to the
// groups in ascending order and the groups are added by a fixed butterfly at the end.
// ------------------------------------------------------------------------------------
template <typename T, int D>
struct RowAcc {
    static constexpr int kE = Pack<T>::kElems;
    static constexpr int kLpr = Tile<T, D>::kChunksPerRow;     // lanes per row
    static constexpr int kGroups = kWave / kLpr;
    float k[kE], v[kE];
    float wsum;                                                // weighted merge only
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < kE; ++i) { k[i] = 0.f; v[i] = 0.f; }
        wsum = 0.f;
    }
    static __device__ __forceinline__ frag_t load_piece(const T* X, int pos, int piece)
    {
        return *reinterpret_cast<const frag_t*>(reinterpret_cast<const char*>(X) + ((size_t)pos * kLpr + piece) * 16);
    }
    // adds a token given its key and value pieces (unit key, raw value); returns the key's
    // norm.  All kLpr lanes of the group must call together.
    __device__ __forceinline__ float accumulate(const frag_t& fk, const frag_t& fv)
    {
        const float ss = group_sum<kLpr>(frag_sumsq<T>(fk));
        const float rn = inv_norm(ss);
        float xk[kE], xv[kE];
        Pack<T>::unpack(fk, xk);
        Pack<T>::unpack(fv, xv);
#pragma unroll
        for (int i = 0; i < kE; ++i) { k[i] = __builtin_fmaf(xk[i], rn, k[i]); v[i] += xv[i]; }
        return sqrtf(ss);
    }
    // the same with weight w >= 0 on the token (score-weighted merge, Sec. 4.2)
    __device__ __forceinline__ float accumulate_weighted(const frag_t& fk, const frag_t& fv, float w)
    {
        const float ss = group_sum<kLpr>(frag_sumsq<T>(fk));
        const float rnw = inv_norm(ss) * w;
        float xk[kE], xv[kE];
        Pack<T>::unpack(fk, xk);
        Pack<T>::unpack(fv, xv);
#pragma unroll
        for (int i = 0; i < kE; ++i) { k[i] = __builtin_fmaf(xk[i], rnw, k[i]); v[i] = __builtin_fmaf(xv[i], w, v[i]); }
        wsum += w;
        return sqrtf(ss);
    }
    // adds the groups together: afterwards every group holds the total
    template <bool kWeighted>
    __device__ __forceinline__ void reduce_groups()
    {
#pragma unroll
        for (int o = kLpr; o < kWave; o <<= 1) {
#pragma unroll
            for (int i = 0; i < kE; ++i) { k[i] += __shfl_xor(k[i], o); v[i] += __shfl_xor(v[i], o); }
            if constexpr (kWeighted) wsum += __shfl_xor(wsum, o);
        }
    }
};

// Adds the members of `target` among `len` listed tokens (destination and position in LDS, ascending)
// to `acc` and returns how many there were; chunks of 64 entries.
template <typename T, int D, bool kWeighted>
__device__ __forceinline__ int gather_members(RowAcc<T, D>& acc, const T* K, const T* V, const float* Wt,
                                              const int* ldest, const int* lpos, int len, int target, int* wlist)
{
    constexpr int kLpr = RowAcc<T, D>::kLpr, kGroups = RowAcc<T, D>::kGroups;
    const int lane = threadIdx.x % kWave;
    const int grp = lane / kLpr, piece = lane % kLpr;
    int count = 0;
    for (int c0 = 0; c0 < len; c0 += kWave) {
        const int i = c0 + lane;
        const bool match = i < len && ldest[i] == target;
        const unsigned long long mask = __ballot(match);
        if (mask == 0ull) continue;                              // wave-uniform
        const int n = __popcll(mask);
        if (match) wlist[__popcll(mask & ((1ull << lane) - 1ull))] = lpos[i];
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        // kInFlight members per lane group at a time, all their loads issued before the first is
        // added; a group still adds its members in ascending order
        constexpr int kInFlight = 4;
        for (int m0 = 0; m0 < n; m0 += kGroups * kInFlight) {
            frag_t fk[kInFlight], fv[kInFlight];
            float w[kInFlight];
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                const int m = m0 + u * kGroups + grp;
                const int pos = m < n ? wlist[m] : 0;
                fk[u] = load_frag_or_zero(K, ((size_t)pos * kLpr + piece) * 16, m < n);
                fv[u] = load_frag_or_zero(V, ((size_t)pos * kLpr + piece) * 16, m < n);
                w[u] = (kWeighted && m < n) ? fmaxf(Wt[pos], 0.f) : 0.f;
            }
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                if (m0 + u * kGroups + grp >= n) break;
                if constexpr (kWeighted) acc.accumulate_weighted(fk[u], fv[u], w[u]);
                else acc.accumulate(fk[u], fv[u]);
            }
        }
        __builtin_amdgcn_wave_barrier();
        count += n;
    }
    return count;
}

// Words that blocks of one launch hand to each other: read and written where every XCD sees them (device scope),
// so that a wait for the stores is all that has to come before the arrival is counted.  A fence would write the whole
// L2 back, with the output rows of every other block: 8 us of a launch whose rows take 10.
__device__ __forceinline__ void store_shared(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float load_shared(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Blocks of a head: first those of the zero class (a.zero_blocks; each takes a stretch of the TBM list,
// a wave an eighth of it), then the output rows, a.rows_per_wave per wave: class-centre slots, then the
// local window.
//
// A centre block first sifts the TBM list: each wave reads an eighth of a piece of it and keeps, in
// order, the tokens that go to one of the block's slots; a slot then looks through the few that were
// kept.  (4032 slots, 4096 tokens, 8 heads, the kernel under a trace: 107 us when every slot walked the whole
// list; 48 with the sift, a shared zero class and one row per 16 lanes in flight, its members' rows requested
// together; 32 now that the zero class's blocks need no fence.)  Several rows per wave where that leaves enough
// blocks, since every block reads the list once.
//
// Several zero-class blocks leave their sums in a.zero_part (the slices' winners, dead by now) and
// count their arrivals on the class's own count, which the last one to arrive overwrites with the
// members' number after adding the blocks' sums in block order.
template <typename T, int D, bool kWeighted>
__global__ __launch_bounds__(kMergeBlock) void merge_kernel(MergeArgs a)
{
    using Acc = RowAcc<T, D>;
    constexpr int kE = Acc::kE, kLpr = Acc::kLpr, kGroups = Acc::kGroups;

    // what was kept of a piece of the TBM list: destination and position
    __shared__ int ldest[kMergeWaves * kMergeStretch];
    __shared__ int lpos[kMergeWaves * kMergeStretch];
    __shared__ int kept_n[kMergeWaves];
    __shared__ int wlist_all[kMergeWaves][kWave];
    __shared__ float zsum[kMergeWaves][2][D];
    __shared__ int zcnt[kMergeWaves];
    __shared__ float zwsum[kMergeWaves];

    const int N = a.seq_len, W = a.window, Nb = a.budget, n_imp = a.n_imp, n_tbm = a.n_tbm;
    const HeadBlock hb = head_block(a.bkv, a.merge_blocks);
    if (hb.head < 0) return;                                // block-uniform
    const int bkv = hb.head, blk = hb.block;
    const T* K = reinterpret_cast<const T*>(a.k) + ((size_t)bkv * N) * D;
    const T* V = reinterpret_cast<const T*>(a.v) + ((size_t)bkv * N) * D;
    T* Ko = reinterpret_cast<T*>(a.k_out) + ((size_t)bkv * (Nb + 1)) * D;
    T* Vo = reinterpret_cast<T*>(a.v_out) + ((size_t)bkv * (Nb + 1)) * D;
    const int32_t* imp = a.imp_idx + (size_t)bkv * n_imp;
    const int32_t* tbm = n_tbm ? a.tbm_idx + (size_t)bkv * n_tbm : nullptr;
    const int32_t* dest = n_tbm ? a.tbm_dest + (size_t)bkv * n_tbm : nullptr;
    int32_t* kept = a.kept_pos + (size_t)bkv * Nb;
    int32_t* cnt = a.slot_count + (size_t)bkv * (n_imp + 1);
    const float* Wt = kWeighted ? a.weight + (size_t)bkv * N : nullptr;

    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int grp = lane / kLpr, piece = lane % kLpr;
    int* wlist = wlist_all[wave];

    const bool zero_class = blk < a.zero_blocks;
    const unsigned long long below = (1ull << lane) - 1ull;
    // Sifts a piece of the list from p0, up to `end`, a stretch (of at most kMergeStretch entries) per wave:
    // the tokens whose destination is in [lo, hi), in order, one list for the block or
    // (own) one per wave in its eighth of the arrays.  `meanwhile` runs while the entries are on their way.
    // Returns the list's length.
    auto sift = [&](int p0, int end, int lo, int hi, bool own, auto meanwhile) {
        const int stretch = min(kMergeStretch, ((end - p0 + kMergeWaves - 1) / kMergeWaves + kWave - 1) / kWave * kWave);
        const int i0 = p0 + wave * stretch, i1 = min(i0 + stretch, end);
        constexpr int kAhead = 8;                            // entries in flight per lane
        static_assert(kMergeStretch == kAhead * kWave, "the longest stretch is one round");
        int d[kAhead], q[kAhead], n = 0;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int i = i0 + u * kWave + lane;
            d[u] = i < i1 ? dest[i] : -1;
            q[u] = i < i1 ? tbm[i] : 0;
        }
        meanwhile();
        int at0 = wave * kMergeStretch, total = 0;
        if (!own) {                                          // block-uniform
#pragma unroll
            for (int u = 0; u < kAhead; ++u) n += __popcll(__ballot(d[u] >= lo && d[u] < hi));
            __syncthreads();                                 // the previous piece is consumed
            if (lane == 0) kept_n[wave] = n;
            __syncthreads();
            at0 = 0;
            for (int w = 0; w < kMergeWaves; ++w) { at0 += w < wave ? kept_n[w] : 0; total += kept_n[w]; }
            n = 0;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const bool in = d[u] >= lo && d[u] < hi;
            const unsigned long long mask = __ballot(in);
            if (in) { const int at = at0 + n + __popcll(mask & below); ldest[at] = d[u]; lpos[at] = clamp_pos(q[u], N); }
            n += __popcll(mask);
        }
        if (!own) __syncthreads();
        return own ? n : total;
    };

    auto nothing = [] {};
    if (zero_class) {
        const int per_block = (n_tbm + a.zero_blocks - 1) / a.zero_blocks;
        const int z0 = min(blk * per_block, n_tbm), z1 = min(z0 + per_block, n_tbm);
        Acc acc; acc.clear();
        int joined = 0;
        for (int p0 = z0; p0 < z1; p0 += kMergeWaves * kMergeStretch) {
            const int n = sift(p0, z1, Nb, Nb + 1, true, nothing);
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            joined += gather_members<T, D, kWeighted>(acc, K, V, Wt, ldest + wave * kMergeStretch, lpos + wave * kMergeStretch, n, Nb, wlist);
            __builtin_amdgcn_wave_barrier();
        }
        // every wave has added its share in order; the waves, then the blocks, are added in order
        acc.template reduce_groups<kWeighted>();
        if (grp == 0) {
#pragma unroll
            for (int i = 0; i < kE; ++i) { zsum[wave][0][piece * kE + i] = acc.k[i]; zsum[wave][1][piece * kE + i] = acc.v[i]; }
        }
        if (lane == 0) { zcnt[wave] = joined; zwsum[wave] = acc.wsum; }
        __syncthreads();
        int total = 0;
        float wtot = 0.f;
        for (int w = 0; w < kMergeWaves; ++w) { total += zcnt[w]; wtot += zwsum[w]; }
        const int tid = threadIdx.x;                         // thread = (key or value, element)
        const int src = tid / D, el = tid % D;
        float sum = 0.f;
        if (src < 2)
            for (int w = 0; w < kMergeWaves; ++w) sum += zsum[w][src][el];
        if (a.zero_blocks > 1) {
            // a record per block: sums of keys and values, members, total weight
            constexpr int kRec = 2 * D + 2;
            float* rec = a.zero_part + ((size_t)bkv * a.zero_stride) + (size_t)blk * kRec;
            if (src < 2) store_shared(rec + tid, sum);
            if (tid == 0) { store_shared(rec + 2 * D, __int_as_float(total)); store_shared(rec + 2 * D + 1, wtot); }
            wait_stores();                                   // every thread's share of the record is out before the block counts as arrived
            __syncthreads();
            if (tid == 0) zcnt[0] = atomicAdd(&cnt[n_imp], 1);
            __syncthreads();
            if (zcnt[0] != a.zero_blocks - 1) return;        // block-uniform: not the last one
            const float* all = a.zero_part + (size_t)bkv * a.zero_stride;
            total = 0; wtot = 0.f; sum = 0.f;
            for (int z = 0; z < a.zero_blocks; ++z) {
                total += __float_as_int(load_shared(all + (size_t)z * kRec + 2 * D));
                wtot += load_shared(all + (size_t)z * kRec + 2 * D + 1);
                if (src < 2) sum += load_shared(all + (size_t)z * kRec + tid);
            }
        }
        const float denom = kWeighted ? wtot : (float)total;     // members, or their total weight
        if (src < 2) {
            const float mean = denom > 0.f ? sum / denom : 0.f;
            (src ? Vo : Ko)[(size_t)Nb * D + el] = (T)mean;
        }
        if (tid == 0) cnt[n_imp] = total;
        return;
    }

    // ---- output rows: rows_per_wave of every wave, the block's being consecutive.  (More than one
    // per wave only where the whole list is one piece: its sifted form then serves all of them.)
    const int rpw = a.rows_per_wave;
    const int block0 = (blk - a.zero_blocks) * kMergeWaves * rpw, job0 = block0 + wave * rpw;
    const int block1 = min(block0 + kMergeWaves * rpw, n_imp);
    constexpr int kPiece = kMergeWaves * kMergeStretch;

    auto local_row = [&](int job) {                          // copied unchanged by one lane group
        const int pos = N - W + (job - n_imp);
        const frag_t fk = Acc::load_piece(K, pos, piece), fv = Acc::load_piece(V, pos, piece);
        *reinterpret_cast<frag_t*>(reinterpret_cast<char*>(Ko) + ((size_t)job * kLpr + piece) * 16) = fk;
        *reinterpret_cast<frag_t*>(reinterpret_cast<char*>(Vo) + ((size_t)job * kLpr + piece) * 16) = fv;
        if (piece == 0) kept[job] = pos;
    };
    // a class-centre slot's row and scalars, by one lane group
    auto write_centre = [&](int job, const Acc& acc, const frag_t& raw_k, const frag_t& raw_v, int c_pos, float c_norm, int members) {
        frag_t out_k = raw_k, out_v = raw_v;                          // nobody joined: exact copy
        const float m = kWeighted ? acc.wsum : (float)members;        // total weight of the entry
        if (members > 1 && m > 0.f) {
            float ok[kE], ov[kE];
#pragma unroll
            for (int i = 0; i < kE; ++i) { ok[i] = c_norm * (acc.k[i] / m); ov[i] = acc.v[i] / m; }
            out_k = Pack<T>::pack(ok);
            out_v = Pack<T>::pack(ov);
        }
        *reinterpret_cast<frag_t*>(reinterpret_cast<char*>(Ko) + ((size_t)job * kLpr + piece) * 16) = out_k;
        *reinterpret_cast<frag_t*>(reinterpret_cast<char*>(Vo) + ((size_t)job * kLpr + piece) * 16) = out_v;
        if (piece == 0) {
            kept[job] = c_pos;
            cnt[job] = members;
            a.k_norm[(size_t)bkv * (n_imp + n_tbm) + job] = c_norm;
        }
    };
    // a slot by the whole wave: the first lane group begins with the centre, every group takes a share of the members
    struct Centre { int pos; frag_t k, v; float w; };
    auto centre_at = [&](int at) {
        Centre c{clamp_pos(at, N), zero_frag(), zero_frag(), 0.f};
        if (grp == 0) {
            c.k = Acc::load_piece(K, c.pos, piece);
            c.v = Acc::load_piece(V, c.pos, piece);
            if constexpr (kWeighted) c.w = fmaxf(Wt[c.pos], 0.f);
        }
        return c;
    };
    auto slot_by_wave = [&](int job, int len, const Centre& c) {
        Acc acc; acc.clear();
        float c_norm = 0.f;
        if (grp == 0) {
            if constexpr (kWeighted) c_norm = acc.accumulate_weighted(c.k, c.v, c.w);
            else c_norm = acc.accumulate(c.k, c.v);
        }
        int joined = 0;
        if (len >= 0) {
            joined = gather_members<T, D, kWeighted>(acc, K, V, Wt, ldest, lpos, len, job, wlist);
        } else {                                             // a list of several pieces: sifted by the block as it goes
            for (int p0 = 0; p0 < n_tbm; p0 += kPiece) {
                const int n = sift(p0, n_tbm, block0, block1, false, nothing);
                if (job < n_imp) joined += gather_members<T, D, kWeighted>(acc, K, V, Wt, ldest, lpos, n, job, wlist);
            }
        }
        acc.template reduce_groups<kWeighted>();
        if (grp == 0 && job < n_imp) write_centre(job, acc, c.k, c.v, c.pos, c_norm, 1 + joined);
    };

    if (n_tbm > kPiece) {                                    // one row per wave; every wave sifts along
        if (block0 < n_imp) {                                // block-uniform
            const int job = job0;
            if (job < n_imp) slot_by_wave(job, -1, centre_at(imp[job]));
            else for (int p0 = 0; p0 < n_tbm; p0 += kPiece) sift(p0, n_tbm, block0, block1, false, nothing);
        }
        if (job0 >= n_imp && job0 < n_imp + W && grp == 0) local_row(job0);
        return;
    }
    if (rpw == 1) {                                          // the wave's centre is fetched beside the list
        const int job = job0, at = job < n_imp ? imp[job] : 0;
        Centre c;
        int len = 0;
        if (block0 < n_imp && n_tbm > 0) len = sift(0, n_tbm, block0, block1, false, [&] { c = centre_at(at); });
        else c = centre_at(at);
        if (job < n_imp) slot_by_wave(job, len, c);
        else if (job < n_imp + W && grp == 0) local_row(job);
        return;
    }
    const int len = block0 < n_imp && n_tbm > 0 ? sift(0, n_tbm, block0, block1, false, nothing) : 0;
    for (int r0 = 0; r0 < rpw; r0 += kGroups) {
        // a row per lane group while slots have few members, else slot after slot
        const int n_rows = min(kGroups, rpw - r0);
        int mine = 0;                                        // members of this lane group's row
        int count[kGroups];
#pragma unroll
        for (int g = 0; g < kGroups; ++g) count[g] = 0;
        for (int c0 = 0; c0 < len; c0 += kWave) {
            const int d = c0 + lane < len ? ldest[c0 + lane] : -1;
#pragma unroll
            for (int g = 0; g < kGroups; ++g) {
                const bool match = d == job0 + r0 + g;
                const unsigned long long mask = __ballot(match);
                const int at = count[g] + __popcll(mask & below);
                if (match && at < kMergeFew) wlist[g * kMergeFew + at] = lpos[c0 + lane];
                count[g] += __popcll(mask);
            }
        }
#pragma unroll
        for (int g = 0; g < kGroups; ++g) mine = g == grp ? count[g] : mine;
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (__any(grp < n_rows && mine > kMergeFew)) {       // wave-uniform
            for (int r = r0; r < r0 + n_rows; ++r) {
                const int job = job0 + r;
                if (job < n_imp) slot_by_wave(job, len, centre_at(imp[job]));
                else if (job < n_imp + W && grp == 0) local_row(job);
            }
            continue;
        }
        const int job = job0 + r0 + grp;
        const bool centre = grp < n_rows && job < n_imp;
        if (grp < n_rows && job >= n_imp && job < n_imp + W) local_row(job);
        Acc acc; acc.clear();
        const int c_pos = centre ? clamp_pos(imp[job], N) : 0;
        const frag_t raw_k = load_frag_or_zero(K, ((size_t)c_pos * kLpr + piece) * 16, centre);
        const frag_t raw_v = load_frag_or_zero(V, ((size_t)c_pos * kLpr + piece) * 16, centre);
        const float c_w = kWeighted && centre ? fmaxf(Wt[c_pos], 0.f) : 0.f;
        // the members, kMergeFew at most; their rows are requested before the first is added
        if (!centre) mine = 0;
        frag_t fk[kMergeFew], fv[kMergeFew];
        float w[kMergeFew];
#pragma unroll
        for (int u = 0; u < kMergeFew; ++u) {
            const int pos = u < mine ? wlist[grp * kMergeFew + u] : 0;
            fk[u] = load_frag_or_zero(K, ((size_t)pos * kLpr + piece) * 16, u < mine);
            fv[u] = load_frag_or_zero(V, ((size_t)pos * kLpr + piece) * 16, u < mine);
            w[u] = kWeighted && u < mine ? fmaxf(Wt[pos], 0.f) : 0.f;
        }
        if (centre) {
            float c_norm;
            if constexpr (kWeighted) c_norm = acc.accumulate_weighted(raw_k, raw_v, c_w);
            else c_norm = acc.accumulate(raw_k, raw_v);
#pragma unroll
            for (int u = 0; u < kMergeFew; ++u)
                if (u < mine) {
                    if constexpr (kWeighted) acc.accumulate_weighted(fk[u], fv[u], w[u]);
                    else acc.accumulate(fk[u], fv[u]);
                }
            write_centre(job, acc, raw_k, raw_v, c_pos, c_norm, 1 + mine);
        }
        __builtin_amdgcn_wave_barrier();                     // the next rows' lists replace these
    }
}

// ------------------------------------------------------------------------------------
// Shared-entry expansion (App. A): one 16-lane group per output row; a merged token's key
// is its entry's key rescaled from the centre's norm to the token's own norm.
// ------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(kMrgBlock) void expand_kernel(ExpandArgs a)
{
    using Acc = RowAcc<T, D>;
    constexpr int kE = Acc::kE, kLpr = Acc::kLpr, kGroups = Acc::kGroups;
    const int n_imp = a.n_imp, n_tbm = a.n_tbm, Nb = a.budget;
    const int n_exp = n_imp + n_tbm + a.window;
    const int bkv = blockIdx.y;
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int grp = lane / kLpr, piece = lane % kLpr;
    const int row = (blockIdx.x * kMrgWaves + wave) * kGroups + grp;
    if (row >= n_exp) return;

    const char* Kc = reinterpret_cast<const char*>(a.k_cache) + (size_t)bkv * (Nb + 1) * D * sizeof(T);
    const char* Vc = reinterpret_cast<const char*>(a.v_cache) + (size_t)bkv * (Nb + 1) * D * sizeof(T);
    char* Ke = reinterpret_cast<char*>(a.k_exp) + ((size_t)bkv * n_exp + row) * D * sizeof(T);
    char* Ve = reinterpret_cast<char*>(a.v_exp) + ((size_t)bkv * n_exp + row) * D * sizeof(T);

    int src = -1, pos = -1;          // cache row the token lives in
    float scale = 1.f;
    bool rescale = false;
    if (row < n_imp) {
        src = row; pos = a.kept_pos[(size_t)bkv * Nb + row];
    } else if (row < n_imp + n_tbm) {
        const int i = row - n_imp;
        const int s = a.tbm_dest[(size_t)bkv * n_tbm + i];
        if (s >= 0 && s < n_imp) {
            const float nc = a.k_norm[(size_t)bkv * (n_imp + n_tbm) + s];
            const float ni = a.k_norm[(size_t)bkv * (n_imp + n_tbm) + n_imp + i];
            src = s; pos = a.tbm_idx[(size_t)bkv * n_tbm + i];
            scale = nc > 0.f ? ni / nc : 0.f;
            rescale = true;
        }
    } else {
        src = n_imp + (row - n_imp - n_tbm); pos = a.kept_pos[(size_t)bkv * Nb + src];
    }
    frag_t fk = zero_frag(), fv = zero_frag();
    if (src >= 0) {
        fk = *reinterpret_cast<const frag_t*>(Kc + ((size_t)src * kLpr + piece) * 16);
        fv = *reinterpret_cast<const frag_t*>(Vc + ((size_t)src * kLpr + piece) * 16);
        if (rescale) {
            float x[kE];
            Pack<T>::unpack(fk, x);
#pragma unroll
            for (int e = 0; e < kE; ++e) x[e] *= scale;
            fk = Pack<T>::pack(x);
        }
    }
    *reinterpret_cast<frag_t*>(Ke + piece * 16) = fk;
    *reinterpret_cast<frag_t*>(Ve + piece * 16) = fv;
    if (piece == 0) a.pos_exp[(size_t)bkv * n_exp + row] = pos;
}

template <typename T, int D>
static hipError_t launch_expand_t(const ExpandArgs& a, hipStream_t st)
{
    const int rows_per_block = kMrgWaves * RowAcc<T, D>::kGroups;
    const int n_exp = a.n_imp + a.n_tbm + a.window;
    dim3 g((n_exp + rows_per_block - 1) / rows_per_block, a.bkv);
    hipLaunchKernelGGL((expand_kernel<T, D>), g, dim3(kMrgBlock), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_expand(const ExpandArgs& a, bool f32, hipStream_t st)
{
    if (f32) {
        if (a.head_dim == 64) return launch_expand_t<float, 64>(a, st);
        return launch_expand_t<float, 128>(a, st);
    }
    if (a.head_dim == 64) return launch_expand_t<bf16_t, 64>(a, st);
    return launch_expand_t<bf16_t, 128>(a, st);
}

// Centre slices per head at most: whole rounds of centres, or, of up to 16 rounds, stages where all blocks are resident even
// so.  The winners of those take 512 KB at most and the norms beside them (256 heads of 4096 centres at most) 4.3 MB, so
// nothing that fitted the fixed scratch of the call without a workspace stops fitting it.  One round is not cut
// (dest_combine_kernel would cost what that gains).
constexpr int kDestResident = 512;
int dest_max_slices(int n_imp, int n_tbm, int bkv, bool f32)
{
    const int stage_rows = f32 ? DestCfg<float>::kStageRows : DestCfg<bf16_t>::kStageRows;
    const int stages = (n_imp + stage_rows - 1) / stage_rows, rounds = (stages + kDestDepth - 1) / kDestDepth;
    if (rounds <= 1) return 1;
    if (rounds > kDestMaxSlices) {
        const int per_slice = (rounds + kDestMaxSlices - 1) / kDestMaxSlices;
        return (rounds + per_slice - 1) / per_slice;
    }
    constexpr int kTile = kMrgWaves * 32;
    const long long lists = std::max(1ll, (long long)((n_tbm + kTile - 1) / kTile) * bkv);
    return std::max(rounds, (int)std::min<long long>(std::min(kDestMaxSlices, stages), kDestResident / lists));
}

// How the centre list is cut: the slices (of whole stages) whose blocks get through soonest, two blocks to a compute
// unit; a block's beginning (two dependent gathers, its tokens' norms) counts as kDestStart stages.  Destination and merge,
// us with 2 / 4 / 8 / 16 slices: 8 heads, 4032 centres, 4096 tokens 75.3 / 60.2 / 63.0 / 70.6; 32 heads of 64, 3968,
// 8000: 426 / 436 / 458 / 506; one head, 2968, 750: 50.2 / 37.5 / 29.9 / 25.7.  The rule's choice: 60, 426 and 25.4; over
// 17 sizes of 1 to 96 heads it is at most 3 % off the best.
constexpr int kDestStart = 4;
static long long dest_cost(long long lists, int stages, int n_slices, int* per_slice)
{
    *per_slice = (stages + n_slices - 1) / n_slices;
    const long long blocks = lists * ((stages + *per_slice - 1) / *per_slice);
    return (blocks + kDestResident - 1) / kDestResident * (*per_slice + kDestStart);
}

template <typename T, int D, int kSim, int kTok>
static hipError_t launch_dest_t(MergeArgs& a, hipStream_t st)
{
    constexpr int kTile = kMrgWaves * 32 * kTok, kStageRows = DestCfg<T>::kStageRows;
    const int tiles = (a.n_tbm + kTile - 1) / kTile, stages = (max(a.n_imp, 1) + kStageRows - 1) / kStageRows;
    const int most = a.n_slices;
    int per = stages;
    if (most > 1) {
        long long best = -1;
        for (int s = 2; s <= most; ++s) {
            int p;
            const long long cost = dest_cost((long long)tiles * a.bkv, stages, s, &p);
            if (best < 0 || cost < best) { best = cost; per = p; }
        }
    }
    a.slice_rows = per * kStageRows;
    a.n_slices = (stages + per - 1) / per;
    const long long grid = head_grid(a.bkv, (long long)tiles * a.n_slices);
    if (grid > 0x7fffffffll) return hipErrorInvalidValue;
    hipLaunchKernelGGL((dest_kernel<T, D, kSim, kTok>), dim3((unsigned)grid), dim3(kMrgBlock), 0, st, a);
    return hipGetLastError();
}

// Token tiles of 64 per wave read every gathered centre row less often; they take over where, with rounds for slices,
// they still make two blocks per compute unit (32 heads, 1436 centres, 1500 tokens: 60 us against 64 with tiles of 32;
// 8 heads, 1984 and 1024: 27.3 against 26.7).  Both sources of the product of
// cosines leave registers for one, float32 rows likewise.
template <typename T, int D, int kSim>
static hipError_t launch_dest(MergeArgs& a, hipStream_t st)
{
    if constexpr (sizeof(T) == 2 && kSim != 2) {
        constexpr int kTile = kMrgWaves * 64, kRound = kDestDepth * DestCfg<T>::kStageRows;
        const long long lists = (long long)((a.n_tbm + kTile - 1) / kTile) * a.bkv;
        if (lists * min(kDestMaxSlices, (a.n_imp + kRound - 1) / kRound) >= kDestResident) return launch_dest_t<T, D, kSim, 2>(a, st);
    }
    return launch_dest_t<T, D, kSim, 1>(a, st);
}

template <typename T, int D>
static hipError_t launch_evict_merge_t(MergeArgs a, hipStream_t st)
{
    hipError_t e = hipSuccess;
    if (a.n_tbm > 0) {
        e = a.similarity == 0 ? launch_dest<T, D, 0>(a, st) : a.similarity == 1 ? launch_dest<T, D, 1>(a, st) : launch_dest<T, D, 2>(a, st);
        if (e != hipSuccess) return e;
        if (a.n_slices > 1) {
            dim3 gc((a.n_tbm + kMrgBlock - 1) / kMrgBlock, a.bkv);
            hipLaunchKernelGGL(dest_combine_kernel, gc, dim3(kMrgBlock), 0, st, a);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    // Rows per wave: as many as leave two blocks per compute unit, where the TBM list is one piece.
    const int jobs = a.n_imp + a.window;
    const long long waves = (long long)jobs * a.bkv;
    a.rows_per_wave = a.n_tbm > kMergeWaves * kMergeStretch ? 1 : (int)std::min<long long>(kMergeMaxRows, std::max<long long>(1, waves / (512 * kMergeWaves)));
    // The zero class is shared by several blocks where the centre list was searched in slices: the
    // winners' array then holds the blocks' sums (2 D + 2 floats per 512 tokens; a slice has one per token).
    a.zero_blocks = a.n_slices > 1 ? std::max(1, a.n_tbm / kZeroTokens) : 1;
    a.zero_part = a.part_best;
    a.zero_stride = (size_t)a.n_slices * a.n_tbm;
    const int per_block = kMergeWaves * a.rows_per_wave;
    a.merge_blocks = a.zero_blocks + (jobs + per_block - 1) / per_block;
    const long long grid = head_grid(a.bkv, a.merge_blocks);
    if (grid > 0x7fffffffll) return hipErrorInvalidValue;
    const dim3 g((unsigned)grid);
    if (a.weight) hipLaunchKernelGGL((merge_kernel<T, D, true>), g, dim3(kMergeBlock), 0, st, a);
    else hipLaunchKernelGGL((merge_kernel<T, D, false>), g, dim3(kMergeBlock), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_evict_merge(const MergeArgs& a, bool f32, hipStream_t st)
{
    if (f32) {
        if (a.head_dim == 64) return launch_evict_merge_t<float, 64>(a, st);
        return launch_evict_merge_t<float, 128>(a, st);
    }
    if (a.head_dim == 64) return launch_evict_merge_t<bf16_t, 64>(a, st);
    return launch_evict_merge_t<bf16_t, 128>(a, st);
}

}  // namespace ems
