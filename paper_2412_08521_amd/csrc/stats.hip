// Per-head statistics of Sec. 4.1: sparsity rate (Eq. 3) and redundancy rate (Eq. 4).
//
// sparsity_kernel    one block per (batch, kv-head): Eq. 2 score of every position, then
//                    the smallest number of top scores whose mass reaches zeta of the total,
//                    found without sorting by an 8-bit-digit radix descent over the
//                    order-preserving integer image of the scores.  Masses are added as
//                    64-bit fixed-point integers, so the result does not depend on the
//                    order in which the atomics land.
// redundancy_stream_kernel  (16-bit) for every token the best key-cosine x value-cosine against
//                    all EARLIER tokens: both cosines as MFMA contractions of raw rows scaled by
//                    reciprocal norms, running maximum per lane, one wave per work item.
// redundancy_kernel  the same for float32 (whose rows fill the registers of a wave, and whose
//                    matrix rate hides the staging), and for the shortest and the longest 16-bit
//                    sequences, in the layout of the merge destination kernel with "centres" = the
//                    causal prefix.
// redundancy_count_kernel  tokens whose best redundancy reaches tau, per head.
#include "ems_common.h"
#include "ems_kernels.h"
#include "ems_rows.h"
#include "ems_stream.h"

namespace ems {

constexpr int kStatBlock = 1024;
constexpr int kStatWaves = kStatBlock / kWave;
constexpr double kMassOne = 1099511627776.0;   // 2^40: fixed-point image of the whole score mass

// scores are >= 0: their bit patterns already order like the values
__device__ __forceinline__ uint32_t score_key(float s) { return __float_as_uint(fmaxf(s, 0.f)); }

constexpr int kSameLanes = 24;                 // lanes on one digit from which one atomic for them all is the cheaper way
constexpr int kStatLds = 32768;                // scores of a head held in LDS (128 KB)

// Sum over the wave, the same in every lane.
__device__ __forceinline__ int wave_add(int v)
{
    v += dpp_i<kDppXor1>(v);
    v += dpp_i<kDppXor2>(v);
    v += dpp_i<kDppHalfMirror>(v);
    v += dpp_i<kDppMirror>(v);
    return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48);
}

// 8 heads of 16384 tokens, calls in a row: 67 us with one thread walking the 256 digits of each pass and every
// walk over the scores reading both arrays; now 32 (under a trace 76 and 45).
__global__ __launch_bounds__(kStatBlock) void sparsity_kernel(StatsArgs a)
{
    __shared__ float kept[kStatLds];
    __shared__ float red[kStatWaves][2];
    __shared__ int cnt[256];
    __shared__ unsigned long long mass[256];
    __shared__ unsigned long long sh_total;
    __shared__ uint32_t sh_prefix;
    __shared__ unsigned long long sh_mass_above;
    __shared__ int sh_count_above;
    __shared__ unsigned long long wave_mass[4];
    __shared__ int wave_cnt[4];

    const int N = a.seq_len;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const float* glo = a.s_glo + (size_t)blockIdx.x * N;
    const float* loc = a.s_loc + (size_t)blockIdx.x * N;

    // Eq. 2 alignment factor, fixed-order sums; kAhead elements' loads in flight per thread
    constexpr int kAhead = 8;
    float sg = 0.f, sl = 0.f;
    for (int j0 = tid; j0 < N; j0 += kStatBlock * kAhead) {
        float g[kAhead], l[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int j = j0 + u * kStatBlock;
            g[u] = j < N ? glo[j] : 0.f;
            l[u] = j < N ? loc[j] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) { sg += g[u]; sl += l[u]; }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) { sg += __shfl_xor(sg, o); sl += __shfl_xor(sl, o); }
    if (lane == 0) { red[wave][0] = sg; red[wave][1] = sl; }
    if (tid == 0) sh_total = 0ull;
    __syncthreads();
    float tot_g = 0.f, tot_l = 0.f;
    for (int w = 0; w < kStatWaves; ++w) { tot_g += red[w][0]; tot_l += red[w][1]; }
    const float align = tot_g > 0.f ? (tot_l / (float)N) / (tot_g / (float)N) : 0.f;

    // Total of the Eq. 2 scores (float tree), then every score as a share of it in fixed point.  The scores
    // stay in LDS where they fit (a thread reads its own elements): the five walks that follow otherwise go back to
    // memory for them.
    const bool in_lds = N <= kStatLds;
    float st = 0.f;
    for (int j0 = tid; j0 < N; j0 += kStatBlock * kAhead) {
        float x[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int j = j0 + u * kStatBlock;
            x[u] = j < N ? fmaxf(glo[j] * align, loc[j]) : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            st += x[u];
            if (in_lds && j0 + u * kStatBlock < N) kept[j0 + u * kStatBlock] = x[u];
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) st += __shfl_xor(st, o);
    __syncthreads();
    if (lane == 0) red[wave][0] = st;
    __syncthreads();
    float tot_s = 0.f;
    for (int w = 0; w < kStatWaves; ++w) tot_s += red[w][0];
    const double to_fixed = tot_s > 0.f ? kMassOne / (double)tot_s : 0.0;

    unsigned long long part = 0ull;
    if (in_lds) {
        for (int j = tid; j < N; j += kStatBlock) part += (unsigned long long)((double)kept[j] * to_fixed);
    } else {
        for (int j0 = tid; j0 < N; j0 += kStatBlock * kAhead) {
            float g[kAhead], l[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int j = j0 + u * kStatBlock;
                g[u] = j < N ? glo[j] : 0.f;
                l[u] = j < N ? loc[j] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) part += (unsigned long long)((double)fmaxf(g[u] * align, l[u]) * to_fixed);
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) part += __shfl_xor(part, o);
    if (lane == 0) atomicAdd(&sh_total, part);
    if (tid == 0) { sh_prefix = 0u; sh_mass_above = 0ull; sh_count_above = 0; }
    __syncthreads();
    // smallest integer mass that counts as "zeta of the total"
    const unsigned long long need_total = (unsigned long long)ceil((double)a.zeta * (double)sh_total);

    for (int shift = 24; shift >= 0; shift -= 8) {
        for (int d = tid; d < 256; d += kStatBlock) { cnt[d] = 0; mass[d] = 0ull; }
        __syncthreads();
        const uint32_t prefix = sh_prefix;
        auto count = [&](float s, bool in) __attribute__((always_inline)) {          // by whole waves
            const uint32_t key = score_key(s);
            bool on = in && (shift == 24 || (key >> ((shift + 8) & 31)) == prefix);
            const int digit = (key >> shift) & 255;
            const unsigned long long q = on ? (unsigned long long)((double)s * to_fixed) : 0ull;
            if (shift == 24) {
                // leading digits are shared: where many lanes agree with the first one, they go into one pair of
                // atomics (the masses' sum in two halves of at most 20 + 6 bits)
                const unsigned long long active = __ballot(on);
                if (active == 0ull) return;                  // wave-uniform
                const int leader = __ffsll((long long)active) - 1;
                const int d0 = __builtin_amdgcn_readlane(digit, leader);
                const bool same = on && digit == d0;
                const int n = __popcll(__ballot(same));
                if (n >= kSameLanes) {                       // wave-uniform
                    const int lo = wave_add(same ? (int)(q & 0xfffffull) : 0), hi = wave_add(same ? (int)(q >> 20) : 0);
                    if (lane == leader) { atomicAdd(&cnt[d0], n); atomicAdd(&mass[d0], (unsigned long long)lo + ((unsigned long long)hi << 20)); }
                    on = on && !same;
                }
            }
            if (on) { atomicAdd(&cnt[digit], 1); atomicAdd(&mass[digit], q); }
        };
        if (in_lds) {
            for (int j0 = 0; j0 < N; j0 += kStatBlock) count(j0 + tid < N ? kept[j0 + tid] : 0.f, j0 + tid < N);
        } else {                                             // from memory: several loads in flight
            constexpr int kFew = 8;
            for (int j0 = tid; j0 - tid < N; j0 += kStatBlock * kFew) {
                float g[kFew], l[kFew];
#pragma unroll
                for (int u = 0; u < kFew; ++u) {
                    const int j = j0 + u * kStatBlock;
                    g[u] = j < N ? glo[j] : 0.f;
                    l[u] = j < N ? loc[j] : 0.f;
                }
#pragma unroll
                for (int u = 0; u < kFew; ++u) count(fmaxf(g[u] * align, l[u]), j0 + u * kStatBlock < N);
            }
        }
        __syncthreads();
        // the digit, from the largest, in which the mass crosses: thread t holds digit 255 - t and the sums
        // of the digits from the top down to it
        const unsigned long long above = sh_mass_above;
        const int count_above = sh_count_above;
        const int d = 255 - min(tid, 255);
        const unsigned long long own = mass[d];
        unsigned long long m_incl = own;
        int c_incl = cnt[d];
        if (tid < 256) {
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const unsigned long long mu = __shfl_up(m_incl, o);
                const int cu = __shfl_up(c_incl, o);
                if (lane >= o) { m_incl += mu; c_incl += cu; }
            }
            if (lane == kWave - 1) { wave_mass[wave] = m_incl; wave_cnt[wave] = c_incl; }
        }
        __syncthreads();
        if (tid < 256) {
            for (int w = 0; w < wave; ++w) { m_incl += wave_mass[w]; c_incl += wave_cnt[w]; }
            const unsigned long long before = above + (m_incl - own);
            const bool crossed = tid > 0 && before >= need_total;        // by a larger digit
            if (!crossed && (above + m_incl >= need_total || d == 0)) {  // one thread
                sh_mass_above = before;
                sh_count_above = count_above + c_incl - cnt[d];
                sh_prefix = (prefix << 8) | (uint32_t)d;
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        // every score with the final key has the same value, hence the same fixed-point mass
        const uint32_t key = sh_prefix;
        const float s_star = __uint_as_float(key);
        const unsigned long long q = (unsigned long long)((double)s_star * to_fixed);
        const int equal = cnt[key & 255];
        const unsigned long long need = need_total > sh_mass_above ? need_total - sh_mass_above : 0ull;
        long long extra = q > 0ull ? (long long)((need + q - 1ull) / q) : (long long)equal;
        if (extra < 1) extra = 1;
        if (extra > equal) extra = equal;
        long long nk = (long long)sh_count_above + extra;
        if (sh_total == 0ull) nk = 1;                        // all scores zero: the first one already "reaches" zeta of 0
        if (nk > N) nk = N;
        if (nk < 1) nk = 1;
        a.p_out[blockIdx.x] = 1.0f - (float)((double)nk / (double)N);
        if (a.n_k_opt) a.n_k_opt[blockIdx.x] = (int32_t)nk;
    }
}

// ------------------------------------------------------------------------------------
constexpr int kRedWaves = 4;
constexpr int kRedBlock = kRedWaves * kWave;
template <typename T> struct RedCfg { static constexpr int kStageRows = 64; };
template <> struct RedCfg<float> { static constexpr int kStageRows = 32; };

// Block = (128 tokens, one (b, kv-head)); each wave keeps 32 tokens' key and value rows in
// registers as MFMA B operands (tokens -> lanes); the earlier tokens stream through LDS as
// the A operands (earlier token -> accumulator register).
template <typename T, int D>
__global__ __launch_bounds__(kRedBlock) void redundancy_kernel(StatsArgs a)
{
    constexpr int kStageRows = RedCfg<T>::kStageRows;
    constexpr int kFrags = Tile<T, D>::kFrags;
    constexpr int kStride = Tile<T, D>::kLdsStride;
    constexpr int kCpr = Tile<T, D>::kChunksPerRow;
    constexpr int kPerThread = kCpr * kStageRows / kRedBlock;

    __shared__ __attribute__((aligned(16))) char lds[2][kStageRows * kStride];
    __shared__ __attribute__((aligned(16))) float lds_rn[2][kStageRows];

    const int N = a.seq_len;
    const int bkv = blockIdx.y;
    const T* src[2] = {reinterpret_cast<const T*>(a.k) + ((size_t)bkv * N) * D,
                       reinterpret_cast<const T*>(a.v) + ((size_t)bkv * N) * D};
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int col = lane & 31, half = lane >> 5;
    // heaviest blocks (latest tokens) first
    const int t_block0 = ((int)gridDim.x - 1 - (int)blockIdx.x) * (kRedWaves * 32);
    const int ti = t_block0 + wave * 32 + col;               // this lane's token
    const bool t_ok = ti < N;

    frag_t bt[2][kFrags];
    float t_rn[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        float ss = 0.f;
#pragma unroll
        for (int f = 0; f < kFrags; ++f) {
            bt[s][f] = load_frag_or_zero(src[s], (size_t)(t_ok ? ti : 0) * Tile<T, D>::kRowBytes + f * 32 + half * 16, t_ok);
            ss += frag_sumsq<T>(bt[s][f]);
        }
        ss += __shfl_xor(ss, 32);
        t_rn[s] = inv_norm(ss);
    }

    float best = -INFINITY;
    const int c_end = min(N, t_block0 + kRedWaves * 32 - 1);  // earlier tokens the block can need
    // the next stage's rows are fetched into registers under the current stage's MFMAs
    frag_t pf[2][kPerThread];
    auto load_rows = [&](int c0) {
#pragma unroll
        for (int i = 0; i < kPerThread; ++i) {
            const int c = threadIdx.x + i * kRedBlock;
            const int ci = c0 + c / kCpr, cc = c % kCpr;
            const bool ok = ci < c_end;
#pragma unroll
            for (int s = 0; s < 2; ++s)
                pf[s][i] = load_frag_or_zero(src[s], ((size_t)(ok ? ci : 0) * kCpr + cc) * 16, ok);
        }
    };
    load_rows(0);
    for (int c0 = 0; c0 < c_end; c0 += kStageRows) {
        __syncthreads();                                   // previous tile fully consumed
#pragma unroll
        for (int i = 0; i < kPerThread; ++i) {
            const int c = threadIdx.x + i * kRedBlock;
            const int row = c / kCpr, cc = c % kCpr;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                *reinterpret_cast<frag_t*>(lds[s] + row * kStride + cc * 16) = pf[s][i];
                const float ss = group_sum<kCpr>(frag_sumsq<T>(pf[s][i]));
                if (cc == 0) lds_rn[s][row] = inv_norm(ss);
            }
        }
        __syncthreads();
        if (c0 + kStageRows < c_end) load_rows(c0 + kStageRows);   // block-uniform
#pragma unroll
        for (int rs = 0; rs < kStageRows / 32; ++rs) {
            const int cbase = c0 + rs * 32;
            if (cbase >= c_end || cbase >= t_block0 + wave * 32 + 31) continue;   // wave-uniform: nothing earlier here
            f32x16_t acc[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                acc[s] = f32x16_t{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int f = 0; f < kFrags; ++f) {
                    const frag_t ac = *reinterpret_cast<const frag_t*>(lds[s] + (rs * 32 + col) * kStride + f * 32 + half * 16);
                    mma<T>(acc[s], ac, bt[s][f]);
                }
            }
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const f32x4_t rk = *reinterpret_cast<const f32x4_t*>(lds_rn[0] + rs * 32 + 8 * q4 + 4 * half);
                const f32x4_t rv = *reinterpret_cast<const f32x4_t*>(lds_rn[1] + rs * 32 + 8 * q4 + 4 * half);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int ci = cbase + 8 * q4 + 4 * half + e;
                    const float r = ((acc[0][4 * q4 + e] * rk[e]) * t_rn[0]) * ((acc[1][4 * q4 + e] * rv[e]) * t_rn[1]);
                    if (ci < ti && r > best) best = r;       // strictly earlier tokens only
                }
            }
        }
    }
    best = fmaxf(best, __shfl_xor(best, 32));                // the other half-wave saw the other rows
    if (half == 0 && t_ok) a.best[(size_t)bkv * N + ti] = best;
}

// ------------------------------------------------------------------------------------
// The 16-bit form.  A wave keeps 32 * kSub tokens' key and value rows in the accumulation registers
// (MFMA B operands, tokens -> lanes) and streams the earlier tokens' rows, 32 of each source per stage,
// through its own LDS ring (A operands, earlier token -> accumulator register); the tokens' lines of
// stages are dealt evenly over the resident waves, and the parts of a token's maximum meet in `best`
// through an integer atomic maximum on the order-preserving image (order-free, hence reproducible).
//
// A round = the two MFMA chains (keys, values) of one token subtile, alternating, with the previous
// subtile's accumulators turned into redundancies in between: (k . k')(v . v') w_j, w_j the reciprocal
// of both norms of the streamed token, two multiplications and half a v_max3 per element; the
// tokens' own norms are applied to the maximum.  The norms of the next stage's rows are formed from
// LDS under the other rounds' chains (64 v_dot2 per stage), since there is no workspace to keep
// them in.  Bound: matrix pipe, 64 MFMAs (2048 clocks) per stage against about 1800 of vector issue.
// 1 x 8 heads of 128, 16384 tokens, 5.5e11 flop, calls in a row with the count: 1585 us with one LDS-staged block
// per 128 tokens (barriers around every stage, nothing in flight), now 537-553 (1.0 PFLOP/s; under a trace, which
// costs this kernel 15 %, 1659 and 629 for the kernel alone).
//
// The short products need norms of a sane size: where |k||v| of a row leaves [2^-30, 2^30] the part is
// redone with every factor applied in turn, as the other form does.
template <int D> struct RedStream { static constexpr int kSub = 4; static constexpr int kRing = D == 128 ? 2 : 4; };

// largest first in integer order; 0 is below the image of every float
__device__ __forceinline__ uint32_t order_image(float x)
{
    const uint32_t b = __float_as_uint(x);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float order_value(uint32_t u)
{
    return u == 0u ? -INFINITY : __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

// a fragment held in the accumulation registers, for the vector ALU
__device__ __forceinline__ frag_t read_acc(const frag_t& b)
{
    frag_t x;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int v;
        asm("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(b[i]));
        x[i] = v;
    }
    return x;
}

__global__ __launch_bounds__(256) void redundancy_clear_kernel(StatsArgs a)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < (size_t)a.bkv * a.seq_len) reinterpret_cast<uint32_t*>(a.best)[i] = 0u;
}

template <int D>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(1, 1))) void redundancy_stream_kernel(StatsArgs a)
{
    using T = bf16_t;
    constexpr int kSub = RedStream<D>::kSub, kRing = RedStream<D>::kRing;
    constexpr int kFrags = Tile<T, D>::kFrags, kRowBytes = Tile<T, D>::kRowBytes, kCpr = Tile<T, D>::kChunksPerRow;
    constexpr int kStageBytes = kStreamRows * kRowBytes;    // one source's rows of a stage
    constexpr int kInstr = kStageBytes / 1024;              // DMA instructions for them
    constexpr int kLoads = 2 * kInstr;
    static_assert(kInstr == 4 || kInstr == 8, "groups of four DMA instructions");
    static_assert((kRing - 1) * kLoads < 64, "vmcnt is a 6-bit counter");
    static_assert((kSub - 1) * kFrags >= 2 * kFrags + 3, "the norms of a stage fit under the chains of its predecessor");
    static_assert(kTrip % kRing == 0, "parts hold whole turns of the ring");
    constexpr int kTokens = 32 * kSub;
    constexpr int kPer = 16 / kFrags;                       // accumulator elements per slot

    __shared__ __attribute__((aligned(1024))) char lds[kRing][2][kStageBytes];
    __shared__ __attribute__((aligned(16))) float lds_w[2][kStreamRows];
    __shared__ float lds_t[2][kTokens];                     // reciprocal norms of the wave's own tokens

    const int N = a.seq_len;
    const DealPass1<kSub> deal(N);
    const DealPlace place = deal_place(a.bkv, a.red_waves);
    if (place.head < 0) return;
    int pos = place.wave * a.red_len;
    const int pos_end = scalar(min(pos + a.red_len, deal.total()));
    const char* K = reinterpret_cast<const char*>(a.k) + (size_t)place.head * N * kRowBytes;
    const char* V = reinterpret_cast<const char*>(a.v) + (size_t)place.head * N * kRowBytes;

    while (pos < pos_end) {
    const int unit = scalar(deal.unit_at(pos));
    const int u0 = deal.first(unit), to = min(pos_end, deal.end(unit));
    const int t0 = scalar(max(pos, u0) - u0);
    const int t1 = scalar(min(to - u0, (min(N, (unit + 1) * kTokens) + kStreamRows - 1) / kStreamRows));
    pos = scalar(to);
    if (t0 >= t1) continue;                                 // before the unit's first stage, or padding
    const int tok0 = unit * kTokens;
    const int t_diag = tok0 / kStreamRows;                  // subtile s is on the diagonal in stage t_diag + s
    // the pipeline takes whole turns of the ring before the diagonal; the diagonal's stages are done one by one
    const int n_pipe = scalar(max(min(t1, t_diag) - t0, 0) / kRing * kRing);

    const int lane = lane_here();
    const int col = lane & 31, half = lane >> 5;

    frag_t bk[kSub][kFrags], bv[kSub][kFrags];
    bool odd_norm = false;                                  // a row whose norms the short products are not made for
#pragma unroll
    for (int s = 0; s < kSub; ++s) {
        const size_t at = (size_t)min(tok0 + s * 32 + col, N - 1) * kRowBytes + half * 16;   // (past the end: any row, its result is not kept)
#pragma unroll
        for (int f = 0; f < kFrags; ++f) {
            bk[s][f] = *reinterpret_cast<const frag_t*>(K + at + f * 32);
            bv[s][f] = *reinterpret_cast<const frag_t*>(V + at + f * 32);
        }
    }
    // only the matrix instructions read the tokens' rows, but for their norms
#pragma unroll
    for (int s = 0; s < kSub; ++s)
#pragma unroll
        for (int f = 0; f < kFrags; ++f) { asm volatile("" : "+a"(bk[s][f])); asm volatile("" : "+a"(bv[s][f])); }
#pragma unroll
    for (int s = 0; s < kSub; ++s) {
        float sk = 0.f, sv = 0.f;
#pragma unroll
        for (int f = 0; f < kFrags; ++f) {
            const frag_t xk = read_acc(bk[s][f]), xv = read_acc(bv[s][f]);
            sk += dot8_bf16(xk, xk);
            sv += dot8_bf16(xv, xv);
            __builtin_amdgcn_sched_barrier(0);
        }
        sk = halves_sum(sk); sv = halves_sum(sv);
        const float rk = inv_norm(sk), rv = inv_norm(sv);
        odd_norm |= (sk > 0.f) & (sv > 0.f) & !((rk * rv >= 0x1p-30f) & (rk * rv <= 0x1p30f));
        lds_t[0][s * 32 + col] = rk; lds_t[1][s * 32 + col] = rv;
    }

    auto swz = [](int row) __attribute__((always_inline)) { return D == 128 ? row & 7 : (row >> 1) & 7; };
    // A row's 16-byte chunks are swizzled within each 128 bytes only: eight lanes read at a time, and a
    // fragment's two places in a 256-byte row stay a constant apart.
    constexpr int kHalfFrags = kFrags < 4 ? kFrags : 4;
    auto dma_src_off = [&](int j, int ln) __attribute__((always_inline)) {
        const int slot = j * kWave + ln, row = slot / kCpr;
        return (unsigned)row * kRowBytes + (unsigned)(((slot % kCpr) ^ swz(row)) << 4);
    };
    // less the offset the instruction itself adds; a second group of four repeats the first 4 KiB on
    // (the swizzle has a period of 16 rows)
    unsigned dma_rel[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) dma_rel[j] = dma_src_off(j, lane) - (unsigned)j * 1024u;
    unsigned frag_base[kHalfFrags];
#pragma unroll
    for (int f = 0; f < kHalfFrags; ++f)
        frag_base[f] = (unsigned)col * kRowBytes + (unsigned)(((f * 2 + half) ^ swz(col)) << 4);
    auto frag_off = [&](int f) __attribute__((always_inline)) { return frag_base[f % kHalfFrags] + (unsigned)(f / kHalfFrags) * 128u; };
    const unsigned lds0 = scalar((int)lds_address(&lds[0][0][0]));

    float raw[kSub];                                        // products that still lack the tokens' own norms
#pragma unroll
    for (int s = 0; s < kSub; ++s) raw[s] = -INFINITY;

    wait_vmem_all_visible();

    if (n_pipe > 0) {
        int t_left = n_pipe;
        const char* k_src = K + (size_t)t0 * kStageBytes;
        const ptrdiff_t v_minus_k = V - K;
        // DMA of the next stage into ring slot `slot`; past the end the last stage again, unread
        auto issue_next = [&](auto slot_c) __attribute__((always_inline)) {
            constexpr int at = decltype(slot_c)::value * 2 * kStageBytes;
            const char* v_src = k_src + v_minus_k;
            static_assert(kInstr == 4 || kRowBytes * 16 == 4096, "the second group's offsets");
            dma_to_lds_x4_at<at>(k_src, dma_rel[0], dma_rel[1], dma_rel[2], dma_rel[3], lds0);
            if constexpr (kInstr > 4) dma_to_lds_x4_at<at + 4096>(k_src + 4096, dma_rel[0], dma_rel[1], dma_rel[2], dma_rel[3], lds0);
            dma_to_lds_x4_at<at + kStageBytes>(v_src, dma_rel[0], dma_rel[1], dma_rel[2], dma_rel[3], lds0);
            if constexpr (kInstr > 4) dma_to_lds_x4_at<at + kStageBytes + 4096>(v_src + 4096, dma_rel[0], dma_rel[1], dma_rel[2], dma_rel[3], lds0);
            advance_cursor<kStageBytes>(t_left, k_src);
        };
        auto rows = [&](int slot, int src, int f) __attribute__((always_inline)) {
            return *reinterpret_cast<const frag_t*>(lds[slot][src] + frag_off(f));
        };
        // The reciprocal of both norms of this lane's row, from the squares this half-wave holds of it (no
        // branches: this runs between matrix instructions).  One reciprocal root of the product has fewer roundings
        // than two rounded roots: the redundancies are 5.6e-8 rms off 64 bits, 6.0e-8 with those (4100 tokens of 128).
        auto both_norms = [&](float sk, float sv) __attribute__((always_inline)) {
            const float k2 = halves_sum(sk), v2 = halves_sum(sv), p = k2 * v2;
            odd_norm |= (k2 > 0.f) & (v2 > 0.f) & !((p >= 0x1p-60f) & (p <= 0x1p60f));
            return p > 0.f ? __builtin_amdgcn_rsqf(p) : 0.f;
        };

        frag_t ak[kFrags], av[kFrags];
        f32x16_t acc[4];                                    // {keys, values} of the present and of the previous subtile
        f32x16_t w_now;
        float w_mine;                                       // this lane's row of the next stage: reciprocal of both norms
        defined_here(acc[0]); defined_here(acc[1]);
        issue_next(ic<0>{});
        issue_next(ic<1>{});
        if constexpr (kRing > 2) { issue_next(ic<2>{}); issue_next(ic<3>{}); }
        wait_vmem<(kRing - 1) * kLoads>();
        {
            float sk = 0.f, sv = 0.f;
#pragma unroll
            for (int f = 0; f < kFrags; ++f) {
                ak[f] = rows(0, 0, f); av[f] = rows(0, 1, f);
                sk += dot8_bf16(ak[f], ak[f]); sv += dot8_bf16(av[f], av[f]);
            }
            w_mine = both_norms(sk, sv);
        }
        // the pipeline starts on a subtile of zeros whose products are no redundancies
#pragma unroll
        for (int r = 0; r < 16; ++r) { acc[2][r] = acc[3][r] = 0.f; w_now[r] = 0.f; }
        bool started = false;                               // false: the first round's maximum is dropped

        auto stage = [&](auto u_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;         // the stage's ring slot
            constexpr int next = (u + 1) % kRing;
            frag_t tmp[2];
            float sk = 0.f, sv = 0.f;
#pragma unroll
            for (int s = 0; s < kSub; ++s) {
                const int ps = (s + kSub - 1) % kSub;       // the previous subtile (of the previous stage when s = 0)
                f32x16_t& accK = acc[2 * (s & 1)];
                f32x16_t& accV = acc[2 * (s & 1) + 1];
                const f32x16_t& prevK = acc[2 * (1 - (s & 1))];
                const f32x16_t& prevV = acc[2 * (1 - (s & 1)) + 1];
                float top = -INFINITY;                      // the first round's result is judged as a whole
                auto weigh = [&](int r0) __attribute__((always_inline)) {
                    float x[kPer];
#pragma unroll
                    for (int e = 0; e < kPer; ++e) x[e] = prevK[r0 + e] * prevV[r0 + e];
#pragma unroll
                    for (int e = 0; e < kPer; ++e) x[e] *= w_now[r0 + e];
#pragma unroll
                    for (int e = 0; e < kPer; ++e) top = fmaxf(top, x[e]);
                };
#pragma unroll
                for (int f = 0; f < kFrags; ++f) {
                    if (f == 0) mma_first<T>(accK, ak[0], bk[s][0]);
                    else mma<T>(accK, ak[f], bk[s][f]);
                    weigh(f * kPer);
                    if (s == kSub - 1) ak[f] = rows(next, 0, f);            // the last chain over this stage's rows
                    __builtin_amdgcn_sched_barrier(0);
                    if (f == 0) mma_first<T>(accV, av[0], bv[s][0]);
                    else mma<T>(accV, av[f], bv[s][f]);
                    if (s == kSub - 1) av[f] = rows(next, 1, f);
                    // the present stage's weights: written by its lanes, read back by accumulator row
                    if (s == 0 && f == 0) lds_w[u & 1][col] = w_mine;
                    // (each half of the registers as soon as the previous stage's last subtile is done with it)
                    if (s == 0 && (f == kFrags / 2 || f == kFrags - 1)) {
#pragma unroll
                        for (int q = f == kFrags / 2 ? 0 : 2; q < (f == kFrags / 2 ? 2 : 4); ++q) {
                            const f32x4_t v = *reinterpret_cast<const f32x4_t*>(&lds_w[u & 1][8 * q + 4 * half]);
#pragma unroll
                            for (int i = 0; i < 4; ++i) w_now[4 * q + i] = v[i];
                        }
                    }
                    // the next stage's norms
                    if (s > 0) {
                        const int q = (s - 1) * kFrags + f;
                        if (q == 0) { wait_vmem<(kRing - 1) * kLoads>(); sk = sv = 0.f; }
                        if (q >= 2 && q < 2 * kFrags + 2) {
                            const frag_t& x = tmp[q % 2];
                            if (q % 2 == 0) sk += dot8_bf16(x, x); else sv += dot8_bf16(x, x);
                        }
                        if (q < 2 * kFrags) tmp[q % 2] = rows(next, q % 2, q / 2);
                        if (q == 2 * kFrags + 2) w_mine = both_norms(sk, sv);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (s == 0) {
                    if (!started) top = -INFINITY;          // wave-uniform
                    started = true;
                    // every row of this stage is in registers: its slot takes the stage a ring ahead
                    issue_next(ic<u>{});
                }
                raw[ps] = fmaxf(raw[ps], top);
            }
        };
        for (int t = 0; t < n_pipe; t += kRing) {
            stage(ic<0>{});
            stage(ic<1>{});
            if constexpr (kRing > 2) { stage(ic<2>{}); stage(ic<3>{}); }
        }
        {   // the last stage's last subtile
            constexpr int at = 2 * ((kSub - 1) & 1);
#pragma unroll
            for (int r = 0; r < 16; ++r) raw[kSub - 1] = fmaxf(raw[kSub - 1], (acc[at][r] * acc[at + 1][r]) * w_now[r]);
        }
        wait_vmem<0>();                                     // no DMA may outlive the wave's LDS
    }

    // the plain form: the diagonal's stages, or everything where a norm is out of its range
    const int lane2 = lane_here(), col2 = lane2 & 31, half2 = lane2 >> 5;
    const bool redo = __any(odd_norm);
    float best[kSub];                                       // finished redundancies
#pragma unroll
    for (int s = 0; s < kSub; ++s) {
        best[s] = -INFINITY;
        if (redo) raw[s] = -INFINITY;
    }
    for (int t = redo ? t0 : t0 + n_pipe; t < t1; ++t) {
        const int row0 = t * kStreamRows;
#pragma unroll
        for (int j = 0; j < kInstr; ++j) {
            const int over = max(row0 + (j * kWave + lane2) / kCpr - (N - 1), 0);      // rows past the end re-read the last row (masked)
            const size_t off = (size_t)(row0 - over) * kRowBytes + dma_src_off(j, lane2);
            *reinterpret_cast<frag_t*>(lds[0][0] + (j * kWave + lane2) * 16) = *reinterpret_cast<const frag_t*>(K + off);
            *reinterpret_cast<frag_t*>(lds[0][1] + (j * kWave + lane2) * 16) = *reinterpret_cast<const frag_t*>(V + off);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        frag_t ak[kFrags], av[kFrags];
        float sk = 0.f, sv = 0.f;
#pragma unroll
        for (int f = 0; f < kFrags; ++f) {
            ak[f] = *reinterpret_cast<const frag_t*>(lds[0][0] + frag_off(f));
            av[f] = *reinterpret_cast<const frag_t*>(lds[0][1] + frag_off(f));
            sk += dot8_bf16(ak[f], ak[f]); sv += dot8_bf16(av[f], av[f]);
        }
        lds_w[0][col2] = inv_norm(halves_sum(sk));
        lds_w[1][col2] = inv_norm(halves_sum(sv));
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int s = 0; s < kSub; ++s) {
            if (row0 < tok0 + s * 32 + 31) {                // wave-uniform: some row is earlier than some token
                f32x16_t accK = zero_acc(), accV = zero_acc();
#pragma unroll
                for (int f = 0; f < kFrags; ++f) { mma<T>(accK, ak[f], bk[s][f]); mma<T>(accV, av[f], bv[s][f]); }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float x = ((accK[r] * lds_w[0][acc_row(r, half2)]) * lds_t[0][s * 32 + col2]) *
                                    ((accV[r] * lds_w[1][acc_row(r, half2)]) * lds_t[1][s * 32 + col2]);
                    if (row0 + acc_row(r, half2) < tok0 + s * 32 + col2) best[s] = fmaxf(best[s], x);
                }
            }
            __builtin_amdgcn_sched_barrier(0);              // one tile's temporaries at a time
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();                    // the next stage's rows may replace these
    }

#pragma unroll
    for (int s = 0; s < kSub; ++s) {
        if (raw[s] > -INFINITY) best[s] = fmaxf(best[s], raw[s] * (lds_t[0][s * 32 + col2] * lds_t[1][s * 32 + col2]));
        best[s] = halves_max(best[s]);  // the half2-waves saw different rows
        const int ti = tok0 + s * 32 + col2;
        if (half2 == 0 && ti < N && best[s] > -INFINITY)
            atomicMax(reinterpret_cast<unsigned int*>(a.best) + (size_t)place.head * N + ti, order_image(best[s]));
    }
    }   // next part
}

// Tokens that reach tau.  After the 16-bit form (red_waves > 0) `best` still holds order images: they are
// turned into the values here.  One block per head, so latency bounds it: with kAhead loads in flight per thread
// 8 heads of 16384 take 5.3 us, one load at a time 11.7.
__global__ __launch_bounds__(kStatBlock) void redundancy_count_kernel(StatsArgs a)
{
    __shared__ int total;
    const int N = a.seq_len;
    float* best = a.best + (size_t)blockIdx.x * N;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    int mine = 0;
    constexpr int kAhead = 8;                                // loads in flight per thread
    for (int j0 = threadIdx.x; j0 < N; j0 += kStatBlock * kAhead) {
        float b[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) b[u] = j0 + u * kStatBlock < N ? best[j0 + u * kStatBlock] : 0.f;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int j = j0 + u * kStatBlock;
            if (j >= N) break;
            if (a.red_waves) { b[u] = order_value(__float_as_uint(b[u])); best[j] = b[u]; }
            mine += b[u] >= a.tau ? 1 : 0;                   // Eq. 4: >=
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mine += __shfl_xor(mine, o);
    if (threadIdx.x % kWave == 0) atomicAdd(&total, mine);
    __syncthreads();
    if (threadIdx.x == 0) a.r_out[blockIdx.x] = (float)((double)total / (double)N);
}

hipError_t launch_sparsity(const StatsArgs& a, hipStream_t st)
{
    hipLaunchKernelGGL(sparsity_kernel, dim3(a.bkv), dim3(kStatBlock), 0, st, a);
    return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_redundancy_t(const StatsArgs& a, hipStream_t st)
{
    const dim3 g((a.seq_len + kRedWaves * 32 - 1) / (kRedWaves * 32), a.bkv);
    hipLaunchKernelGGL((redundancy_kernel<T, D>), g, dim3(kRedBlock), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(redundancy_count_kernel, dim3(a.bkv), dim3(kStatBlock), 0, st, a);
    return hipGetLastError();
}

constexpr int kRedStreamMax = 1 << 21;      // a head's line of stages is counted in 32 bits: longer sequences take the other form

// Up to this length the other form takes the 16-bit rows as well: a wave of the stream begins with 8 us of loads and
// norms, and one more launch clears `best`.  (us, stream / blocks.  128: 1 head of 350 24.7 / 22.4, of 450 24.7 /
// 27.9; 128 heads of 450 40.8 / 34.0, of 513 42.4 / 51.1; 1100 of 256 103 / 89, of 385 183 / 225.  64: 1 head of 450 21.4 / 20.0, of
// 600 21.6 / 24.3; 128 heads of 700 39.6 / 33.6, of 900 49.0 / 59.1; 1100 of 700 227 / 190, of 900 330 / 402.)
static int red_block_max(int head_dim, int heads)
{
    if (head_dim == 64) return heads <= 16 ? 512 : 768;
    return heads <= 16 ? 384 : heads <= 128 ? 448 : 256;
}

template <int D>
static hipError_t launch_redundancy_stream(StatsArgs a, hipStream_t st)
{
    if (a.seq_len > kRedStreamMax || a.seq_len <= red_block_max(D, a.bkv)) return launch_redundancy_t<bf16_t, D>(a, st);
    const DealPass1<RedStream<D>::kSub> deal(a.seq_len);
    deal_over_waves(1024, a.bkv, deal.total(), kTrip, kTrip, &a.red_len, &a.red_waves);
    const long long grid = deal_grid(a.bkv, a.red_waves), clear = ((long long)a.bkv * a.seq_len + 255) / 256;
    if (grid > 0x7fffffffll || clear > 0x7fffffffll) return hipErrorInvalidValue;
    hipLaunchKernelGGL(redundancy_clear_kernel, dim3((unsigned)clear), dim3(256), 0, st, a);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL((redundancy_stream_kernel<D>), dim3((unsigned)grid), dim3(kWave), 0, st, a);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL(redundancy_count_kernel, dim3(a.bkv), dim3(kStatBlock), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_redundancy(const StatsArgs& a, bool f32, hipStream_t st)
{
    if (f32) return a.head_dim == 64 ? launch_redundancy_t<float, 64>(a, st) : launch_redundancy_t<float, 128>(a, st);
    return a.head_dim == 64 ? launch_redundancy_stream<64>(a, st) : launch_redundancy_stream<128>(a, st);
}

}  // namespace ems
