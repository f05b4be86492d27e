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
#include "ems_red_weights.h"
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
// tokens' own norms are applied to the maximum.  The streamed rows' norms are formed at the start of their stage,
// since there is no workspace to keep them in.  Bound: matrix pipe, 144 MFMAs (2304 clocks) per stage against about
// 2100 of issue.
// 1 x 8 heads of 128, 16384 tokens, 5.5e11 flop, calls in a row with the count, us: 1585 with one LDS-staged block
// per 128 tokens (barriers around every stage, nothing in flight); 517-533 as a stream of 32x32x16 products with the norms by
// v_dot2 and the diagonal's stages one by one; 437-445 now (1.26 PFLOP/s; without the streamed rows' DMA, which costs
// issue slots and the L2's misses, 391; 290 for the products alone).  4 heads of 32768: 1006-1040, now 872-899; 8 heads of 16384, size
// 64: 319-332, now 251.
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

__device__ __forceinline__ f32x4_t zero4() { return f32x4_t{0.f, 0.f, 0.f, 0.f}; }

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
    constexpr int kFrags = D / 32;                          // 32 elements of a row are one fragment of four lanes
    constexpr int kRowBytes = Tile<T, D>::kRowBytes, kCpr = Tile<T, D>::kChunksPerRow;
    constexpr int kStageBytes = kStreamRows * kRowBytes;    // one source's rows of a stage
    constexpr int kInstr = kStageBytes / 1024;              // DMA instructions for them
    constexpr int kLoads = 2 * kInstr;
    static_assert(kInstr == 4 || kInstr == 8, "groups of four DMA instructions");
    static_assert((kRing - 1) * kLoads < 64, "vmcnt is a 6-bit counter");
    static_assert(kTrip % kRing == 0 && kSub == kTrip, "parts hold whole turns of the ring, the diagonal is a trip");
    constexpr int kTokens = 32 * kSub;
    // A subtile's round: kProducts matrix instructions with 24 ticks of vector work evenly between them (an instruction
    // that finds the matrix pipe busy holds up what is behind it): for each of 8 pairs of the previous subtile's
    // elements one to multiply keys by values, one to apply the weights, one for the maximum.  The first round of a
    // stage is preceded by its rows' squares.
    constexpr int kProducts = 8 * kFrags, kSquares = 4 * kFrags, kTicks = 24;

    __shared__ __attribute__((aligned(1024))) char lds[kRing][2][kStageBytes];
    static_assert(RedWeights::sound() && RedWeights::kRows == kStreamRows && RedWeights::kLanes == kWave, "the weights' places");
    __shared__ __attribute__((aligned(16))) float lds_w[2][RedWeights::kFloats];
    __shared__ float lds_t[3][kTokens];                     // reciprocal norms of the wave's own tokens: key, value, both

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
    // the pipeline takes the stages before the diagonal and the diagonal's own, each a whole number of turns of the ring
    // (parts are whole trips)
    const int n_int = scalar(max(min(t1, t_diag) - t0, 0));
    const bool on_diag = t1 > t_diag;                       // wave-uniform

    const int lane = lane_here();
    const int col = lane % 16, group = lane / 16;           // in an operand: its row, the row's chunk (modulo the groups)

    frag_t bk[kSub][2][kFrags], bv[kSub][2][kFrags];
    bool odd_norm = false;                                  // a row whose norms the short products are not made for
#pragma unroll
    for (int s = 0; s < kSub; ++s)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const size_t at = (size_t)min(tok0 + s * 32 + j * 16 + col, N - 1) * kRowBytes + group * 16;   // (past the end: any row, its result is not kept)
#pragma unroll
            for (int f = 0; f < kFrags; ++f) {
                bk[s][j][f] = *reinterpret_cast<const frag_t*>(K + at + f * 64);
                bv[s][j][f] = *reinterpret_cast<const frag_t*>(V + at + f * 64);
            }
        }
    // only the matrix instructions read the tokens' rows, but for their norms
#pragma unroll
    for (int s = 0; s < kSub; ++s)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int f = 0; f < kFrags; ++f) { asm volatile("" : "+a"(bk[s][j][f])); asm volatile("" : "+a"(bv[s][j][f])); }
#pragma unroll
    for (int s = 0; s < kSub; ++s)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float sk = 0.f, sv = 0.f;
#pragma unroll
            for (int f = 0; f < kFrags; ++f) {
                const frag_t xk = read_acc(bk[s][j][f]), xv = read_acc(bv[s][j][f]);
                sk += dot8_bf16(xk, xk);
                sv += dot8_bf16(xv, xv);
                __builtin_amdgcn_sched_barrier(0);
            }
            sk = quarters_sum(sk); sv = quarters_sum(sv);
            const float rk = inv_norm(sk), rv = inv_norm(sv);
            odd_norm |= (sk > 0.f) & (sv > 0.f) & !((rk * rv >= 0x1p-30f) & (rk * rv <= 0x1p30f));
            lds_t[0][s * 32 + j * 16 + col] = rk; lds_t[1][s * 32 + j * 16 + col] = rv;
            // (one root of the product, with a Newton step: the redundancies are 5.15e-8 rms off 64 bits at 4100 tokens of 128,
            // 4.41e-8 of 64; 5.55e-8 and 5.03e-8 where the two roots were multiplied)
            lds_t[2][s * 32 + j * 16 + col] = sk * sv > 0.f ? row_inv_norm<float>(sk * sv) : 0.f;
        }

    // (sixteen lanes read at a time: the chunks of sixteen rows lie in different banks)
    auto swz = [](int row) __attribute__((always_inline)) { return swz_key<T, D>(row); };
    auto dma_src_off = [&](int j, int ln) __attribute__((always_inline)) {
        const int slot = j * kWave + ln, row = slot / kCpr;
        return (unsigned)row * kRowBytes + (unsigned)(((slot % kCpr) ^ swz(row)) << 4);
    };
    // less the offset the instruction itself adds; a second group of four repeats the first 4 KiB on
    // (the swizzle has a period of 16 rows)
    unsigned dma_rel[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) dma_rel[j] = dma_src_off(j, lane) - (unsigned)j * 1024u;
    unsigned frag_base[kFrags];
#pragma unroll
    for (int f = 0; f < kFrags; ++f)
        frag_base[f] = (unsigned)col * kRowBytes + (unsigned)(((f * 4 + group) ^ swz(col)) << 4);
    auto frag_off = [&](int i, int f) __attribute__((always_inline)) { return frag_base[f] + (unsigned)(i * 16) * kRowBytes; };   // (rows 16 apart are swizzled alike)
    const unsigned lds0 = scalar((int)lds_address(&lds[0][0][0]));

    float raw[kSub][2];                                // products that still lack the tokens' own norms
#pragma unroll
    for (int s = 0; s < kSub; ++s)
#pragma unroll
        for (int j = 0; j < 2; ++j) raw[s][j] = -INFINITY;

    wait_vmem_all_visible();

    if (n_int > 0 || on_diag) {
        const bool whole = (unit + 1) * kTokens <= N;       // the diagonal's rows all exist: its first ones follow in the stream
        int t_left = n_int + (on_diag && whole ? kRing : 0);
        const char* k_src = K + (size_t)t0 * kStageBytes;
        const ptrdiff_t v_minus_k = V - K;
        // One DMA instruction (of kLoads) of the next stage into ring slot `slot`; past the end the last stage again, unread
        auto issue_one = [&](auto slot_c, auto n_c) __attribute__((always_inline)) {
            constexpr int n = decltype(n_c)::value, src = n / kInstr, j = n % kInstr;
            constexpr int at = (decltype(slot_c)::value * 2 + src) * kStageBytes + j / 4 * 4096;
            static_assert(kInstr == 4 || kRowBytes * 16 == 4096, "the second group's offsets");
            dma_one_to_lds_at<at, j % 4 * 1024>(k_src + (src ? v_minus_k : 0) + j / 4 * 4096, dma_rel[j % 4], lds0);
            if constexpr (n == kLoads - 1) advance_cursor<kStageBytes>(t_left, k_src);
        };
        auto issue_next = [&](auto slot_c) __attribute__((always_inline)) {
            issue_one(slot_c, ic<0>{}); issue_one(slot_c, ic<1>{}); issue_one(slot_c, ic<2>{}); issue_one(slot_c, ic<3>{});
            issue_one(slot_c, ic<4>{}); issue_one(slot_c, ic<5>{}); issue_one(slot_c, ic<6>{}); issue_one(slot_c, ic<7>{});
            if constexpr (kLoads > 8) {
                issue_one(slot_c, ic<8>{}); issue_one(slot_c, ic<9>{}); issue_one(slot_c, ic<10>{}); issue_one(slot_c, ic<11>{});
                issue_one(slot_c, ic<12>{}); issue_one(slot_c, ic<13>{}); issue_one(slot_c, ic<14>{}); issue_one(slot_c, ic<15>{});
            }
        };
        // The same for the diagonal's stage d; rows past the end re-read the last row (only tokens past it are later)
        auto issue_diag = [&](int d, int slot, int n) __attribute__((always_inline)) {
            const int ln = lane_here(), j = n % kInstr, row0 = min(tok0 + d * kStreamRows, N - 1);
            const int row = (j * kWave + ln) / kCpr, at = min(tok0 + d * kStreamRows + row, N - 1) - row0;
            dma_to_lds<16>((n < kInstr ? K : V) + (size_t)row0 * kRowBytes, dma_src_off(j, ln) + (unsigned)((at - row) * kRowBytes),
                           lds0 + (slot * 2 + n / kInstr) * kStageBytes + j * 1024);
        };
        auto rows = [&](int slot, int src, int i, int f) __attribute__((always_inline)) {
            return *reinterpret_cast<const frag_t*>(lds[slot][src] + frag_off(i, f));
        };
        frag_t ak[2][kFrags], av[2][kFrags];
        f32x4_t accs[2][2][2][2];                           // [present / previous subtile][keys, values][streamed rows][tokens]
        f32x4_t w[2][2];                                    // the weights by accumulator row, of this stage and the last
        // A row's squares are the diagonal of its tile's product with itself: 16 matrix instructions a stage.
        // (By v_dot2, 64 of them, which wait for the matrix pipe to drain and hold up its next instruction, 16
        // clocks each time: 16384 tokens, 8 heads of 128, 505 us.)  Subnormal squares are kept either way: with square sums of
        // 2^-128 to 2^-136 the redundancies are as close to 64 bits as the block form's.
        f32x4_t square[2][2];                               // [keys, values][streamed rows]
        const bool diag = RedWeights::holds(lane);          // this lane has row col's, in register col % 4
        const int w_at = RedWeights::slot(lane);
        // the pipeline starts on a subtile of zeros whose products are no redundancies
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int j = 0; j < 2; ++j) accs[1][0][i][j] = accs[1][1][i][j] = zero4();
            w[1][i] = zero4();
        }
        bool started = false;                               // false: the first round's maximum is dropped

        // rows of the diagonal tile that are earlier than the lane's token
        bool earlier[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) earlier[r] = 4 * group + r < col;

        auto dma_at = [&](auto slot_c, int n) __attribute__((always_inline)) {
            switch (n) {                                    // (a constant once the loops are unrolled)
            case 0: issue_one(slot_c, ic<0>{}); break;
            case 1: issue_one(slot_c, ic<1>{}); break;
            case 2: issue_one(slot_c, ic<2>{}); break;
            case 3: issue_one(slot_c, ic<3>{}); break;
            case 4: issue_one(slot_c, ic<4>{}); break;
            case 5: issue_one(slot_c, ic<5>{}); break;
            case 6: issue_one(slot_c, ic<6>{}); break;
            case 7: issue_one(slot_c, ic<7>{}); break;
            default: if constexpr (kLoads > 8) {
                switch (n) {
                case 8: issue_one(slot_c, ic<8>{}); break;
                case 9: issue_one(slot_c, ic<9>{}); break;
                case 10: issue_one(slot_c, ic<10>{}); break;
                case 11: issue_one(slot_c, ic<11>{}); break;
                case 12: issue_one(slot_c, ic<12>{}); break;
                case 13: issue_one(slot_c, ic<13>{}); break;
                case 14: issue_one(slot_c, ic<14>{}); break;
                default: issue_one(slot_c, ic<15>{}); break;
                }
            }
            }
        };

        auto stage = [&](auto u_c, auto d_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;         // the stage's ring slot
            constexpr int d = decltype(d_c)::value;         // its rows are subtile d's own (-1: earlier than all)
            constexpr int next = (u + 1) % kRing;
            float x[2], p[2], x2 = 0.f;
            // What the products of the first round leave time for: the reciprocal of both norms, one reciprocal root of
            // the product, which has fewer roundings than two rounded roots.  No branches: this runs between matrix
            // instructions.
            auto norm_step = [&](int n) __attribute__((always_inline)) {
                auto pick = [&](const f32x4_t& v) __attribute__((always_inline)) {
                    const float lo = col & 1 ? v[1] : v[0], hi = col & 1 ? v[3] : v[2];
                    return col & 2 ? hi : lo;
                };
                const int i = n / 4, part = n % 4;
                if (n < 8) {
                    if (part == 0) p[i] = pick(square[0][i]);
                    if (part == 1) x2 = pick(square[1][i]);
                    if (part == 2) {
                        const float k2 = p[i];
                        p[i] *= x2;
                        odd_norm |= diag & (k2 > 0.f) & (x2 > 0.f) & !((p[i] >= 0x1p-60f) & (p[i] <= 0x1p60f));
                    }
                    if (part == 3) p[i] = p[i] > 0.f ? __builtin_amdgcn_rsqf(p[i]) : 0.f;
                }
                // written by accumulator column, read back by row
                if (n == 8) { lds_w[u & 1][w_at] = p[0]; lds_w[u & 1][w_at + RedWeights::kSecond] = p[1]; }
                if (n == 9) {
#pragma unroll
                    for (int i2 = 0; i2 < 2; ++i2) w[u & 1][i2] = *reinterpret_cast<const f32x4_t*>(&lds_w[u & 1][16 * i2 + 4 * group]);
                }
            };
#pragma unroll
            for (int s = 0; s < kSub; ++s) {
                const int ps = (s + kSub - 1) % kSub;       // the previous subtile (of the previous stage when s = 0)
                auto& now = accs[s & 1];
                auto& prev = accs[1 - (s & 1)];
                const auto& pw = w[s == 0 ? 1 - (u & 1) : u & 1];
                float top[2] = {-INFINITY, -INFINITY};      // the first round's result is judged as a whole
                auto tick = [&](int k) __attribute__((always_inline)) {
                    const int e = k / 3, phase = k % 3, j = e / 4, r = e % 4;       // pair e: two rows' elements of one token
                    if (s > 0 && ps < d) return;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        if (s > 0 && ps == d && phase == 2) x[i] = i < j || (i == j && earlier[r]) ? x[i] : -INFINITY;
                        if (phase == 0) x[i] = prev[0][i][j][r] * prev[1][i][j][r];
                        if (phase == 1) x[i] *= pw[i][r];
                    }
                    if (phase == 2) top[j] = fmaxf(fmaxf(top[j], x[0]), x[1]);
                };
                if (s == 0) {
#pragma unroll
                    for (int m = 0; m < kSquares; ++m) {
                        const int f = m / 4, src = m / 2 % 2, i = m % 2;
                        const frag_t& y = (src ? av : ak)[i][f];
                        square[src][i] = mma16(y, y, f == 0 ? zero4() : square[src][i]);
#pragma unroll
                        for (int k = m * kTicks / kSquares; k < (m + 1) * kTicks / kSquares; ++k) tick(k);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                // the next stage has landed
                constexpr int kOfNext = (kSub - 1) * kLoads / kSub;         // of the stage a ring ahead, by now
                constexpr int kAhead = d < 0 ? kRing - 2 : (d + kRing < kSub ? kRing : kSub - d) - 2;
                if (s == kSub - 1 && d < kSub - 1) wait_vmem<(kAhead < 0 ? 0 : kAhead) * kLoads + (d + kRing < kSub ? kOfNext : 0)>();
#pragma unroll
                for (int m = 0; m < kProducts; ++m) {
                    // (each shares an operand with the one before)
                    const int f = m / 8, src = m / 4 % 2, j = m / 2 % 2, i = j ? 1 - m % 2 : m % 2;
                    frag_t (&a_src)[2][kFrags] = src ? av : ak;
                    if (s >= d) now[src][i][j] = mma16(a_src[i][f], (src ? bv : bk)[s][j][f], f == 0 ? zero4() : now[src][i][j]);
                    if (s == 0) {
#pragma unroll
                        for (int n = m * 20 / kProducts; n < (m + 1) * 20 / kProducts; ++n) if (n >= 2 && n < 12) norm_step(n - 2);
                    } else {
#pragma unroll
                        for (int k = m * kTicks / kProducts; k < (m + 1) * kTicks / kProducts; ++k) tick(k);
                    }
                    if (s == kSub - 1 && j == 1) a_src[i][f] = rows(next, src, i, f);      // the last chain over this stage's rows
                    // Every row of this stage is in registers once their squares are: its slot takes the stage a ring
                    // ahead, an instruction at a time
                    // (four in a row wait for each other: 455 us against 446)
                    if (m % 8 == 4) {
                        if (d < 0) dma_at(ic<u>{}, s * (kLoads / kSub) + m / 8);
                        else if (d + kRing < kSub) issue_diag(d + kRing, u, s * (kLoads / kSub) + m / 8);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    if (s == 0 && !started) top[j] = -INFINITY;        // wave-uniform
                    raw[ps][j] = fmaxf(raw[ps][j], top[j]);
                }
                if (s == 0) started = true;
            }
        };
        auto first_rows = [&]() __attribute__((always_inline)) {        // of ring slot 0
            wait_vmem<(kRing - 1) * kLoads>();
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int f = 0; f < kFrags; ++f) { ak[i][f] = rows(0, 0, i, f); av[i][f] = rows(0, 1, i, f); }
        };
        if (n_int > 0) {
            issue_next(ic<0>{});
            issue_next(ic<1>{});
            if constexpr (kRing > 2) { issue_next(ic<2>{}); issue_next(ic<3>{}); }
            first_rows();
            for (int t = 0; t < n_int; t += kRing) {
                stage(ic<0>{}, ic<-1>{});
                stage(ic<1>{}, ic<-1>{});
                if constexpr (kRing > 2) { stage(ic<2>{}, ic<-1>{}); stage(ic<3>{}, ic<-1>{}); }
            }
        }
        if (on_diag) {
            if (n_int == 0 || !whole) {                     // they do not follow in the stream
                wait_vmem<0>();
#pragma unroll
                for (int t = 0; t < kRing; ++t)
#pragma unroll
                    for (int n = 0; n < kLoads; ++n) issue_diag(t, t, n);
                first_rows();
            }
            stage(ic<0>{}, ic<0>{});
            stage(ic<1>{}, ic<1>{});
            stage(ic<2 % kRing>{}, ic<2>{});
            stage(ic<3 % kRing>{}, ic<3>{});
        }
        // the last stage's last subtile
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float y = (accs[1][0][i][j][r] * accs[1][1][i][j][r]) * w[1][i][r];
                    const bool seen = !on_diag || i < j || (i == j && earlier[r]);
                    raw[kSub - 1][j] = fmaxf(raw[kSub - 1][j], seen ? y : -INFINITY);
                }
        wait_vmem<0>();                                     // no DMA may outlive the wave's LDS
    }

    // the plain form, where a norm is out of its range
    const int lane2 = lane_here(), col2 = lane2 % 16, group2 = lane2 / 16;
    const bool redo = __any(odd_norm);
    float best[kSub][2];                               // finished redundancies
#pragma unroll
    for (int s = 0; s < kSub; ++s)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            best[s][j] = -INFINITY;
            if (redo) raw[s][j] = -INFINITY;
        }
    for (int t = redo ? t0 : t1; t < t1; ++t) {
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
        frag_t ak[2][kFrags], av[2][kFrags];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            float sk = 0.f, sv = 0.f;
#pragma unroll
            for (int f = 0; f < kFrags; ++f) {
                ak[i][f] = *reinterpret_cast<const frag_t*>(lds[0][0] + frag_off(i, f));
                av[i][f] = *reinterpret_cast<const frag_t*>(lds[0][1] + frag_off(i, f));
                sk += dot8_bf16(ak[i][f], ak[i][f]); sv += dot8_bf16(av[i][f], av[i][f]);
            }
            lds_w[0][i * 16 + col2] = inv_norm(quarters_sum(sk));
            lds_w[1][i * 16 + col2] = inv_norm(quarters_sum(sv));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int s = 0; s < kSub; ++s) {
            if (row0 < tok0 + s * 32 + 31) {                // wave-uniform: some row is earlier than some token
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        f32x4_t accK = zero4(), accV = zero4();
#pragma unroll
                        for (int f = 0; f < kFrags; ++f) {
                            accK = mma16(ak[i][f], bk[s][j][f], accK);
                            accV = mma16(av[i][f], bv[s][j][f], accV);
                        }
                        const int tok = s * 32 + j * 16 + col2;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int row = i * 16 + 4 * group2 + r;
                            const float x = ((accK[r] * lds_w[0][row]) * lds_t[0][tok]) * ((accV[r] * lds_w[1][row]) * lds_t[1][tok]);
                            if (row0 + row < tok0 + tok) best[s][j] = fmaxf(best[s][j], x);
                        }
                    }
            }
            __builtin_amdgcn_sched_barrier(0);              // one tile's temporaries at a time
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();                    // the next stage's rows may replace these
    }

#pragma unroll
    for (int s = 0; s < kSub; ++s)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int tok = s * 32 + j * 16 + col2, ti = tok0 + tok;
            float b = best[s][j];
            if (raw[s][j] > -INFINITY) b = fmaxf(b, raw[s][j] * lds_t[2][tok]);
            b = quarters_max(b);                                  // the groups saw different rows
            if (group2 == 0 && ti < N && b > -INFINITY)
                atomicMax(reinterpret_cast<unsigned int*>(a.best) + (size_t)place.head * N + ti, order_image(b));
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
// norms, and one more launch clears `best`.  (us, stream / blocks.  128: 1 head of 256 17.0 / 17.7, of 200 16.7 / 15.9;
// 128 heads of 300 25.6 / 23.3, of 384 25.5 / 27.1; 1100 of 128 40.0 / 37.0, of 200 66.8 / 76.4.  64: 1 head of 256 14.7 /
// 13.3, of 384 15.0 / 17.3; 128 heads of 300 19.5 / 16.7, of 384 18.6 / 18.9; 1100 of 300 59.7 / 57.6, of 384 60.6 / 64.3.)
static int red_block_max(int head_dim, int heads)
{
    if (head_dim == 64) return heads <= 16 ? 288 : 352;
    return heads <= 16 ? 256 : heads <= 128 ? 352 : 160;
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
