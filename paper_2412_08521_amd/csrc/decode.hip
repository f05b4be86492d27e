// Decode-time update of the compressed cache (Sec. 3.3, decoding paragraph; App. A,
// "Evict-then-Merge Details").
//
// decode_init_kernel  builds the per-token table (position, cache row, key norm, s_Glo,
//                     s_Loc^past, s_Loc^cur) from what the prefill compression returned.
// decode_step_kernel  one generated token: one block per (batch, kv-head) runs the whole
//                     step (for large caches it is three or four launches, all but one over slices of the table or
//                     of the cache rows: decode_logits_kernel, decode_choose_kernel, decode_commit_kernel, kPart) -- attention row of the new query over the expanded run-time
//                     cache (one dot product per cache ROW, shared by the tokens that share
//                     the entry; coalesced row loads, v_dot2 partials added with DPP),
//                     score accumulation, window ring shift, least important centre, its
//                     most similar centre, merge-or-evict with the look-up-table remap, new
//                     centre, past/cur swap.  Phases are separated by block barriers that
//                     every thread reaches.
#include "ems_common.h"
#include "ems_kernels.h"
#include "ems_rows.h"

namespace ems {

// ---- wave and block reductions.  Inside a wave the combine runs on DPP lane permutations
// (xor 1, xor 2 inside quads, then the half-row and row mirrors), which have ALU latency;
// the four row results are then read through scalar registers, so the result is uniform.
// all 16 lanes of every row end up with their row's result
template <bool kMax>
__device__ __forceinline__ float row_reduce(float v)
{
    v = comb<kMax>(v, dpp_f<kDppXor1>(v));
    v = comb<kMax>(v, dpp_f<kDppXor2>(v));
    v = comb<kMax>(v, dpp_f<kDppHalfMirror>(v));
    v = comb<kMax>(v, dpp_f<kDppMirror>(v));
    return v;
}
template <bool kMax>
__device__ __forceinline__ float wave_reduce(float v)
{
    v = row_reduce<kMax>(v);
    return comb<kMax>(comb<kMax>(lane_value(v, 0), lane_value(v, 16)), comb<kMax>(lane_value(v, 32), lane_value(v, 48)));
}

// The softmax state (reference m, sum l of the weights relative to it) of G rows over the block, and two plain totals with it:
// one barrier for what a maximum, a sum and the totals would take two each for.  (`buf` is the call's own.)  The result is identical in
// every thread.
template <int kWaves, int G>
__device__ __forceinline__ void block_softmax(float (&m)[G], float (&l)[G], float (&tot)[2], float (*buf)[kWaves])
{
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    float top[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        top[g] = wave_reduce<true>(m[g]);
        l[g] = wave_reduce<false>(m[g] > -INFINITY ? l[g] * exp2_fast(m[g] - top[g]) : 0.f);
    }
    tot[0] = wave_reduce<false>(tot[0]);
    tot[1] = wave_reduce<false>(tot[1]);
    if (lane == 0) {
#pragma unroll
        for (int g = 0; g < G; ++g) { buf[g][wave] = top[g]; buf[G + g][wave] = l[g]; }
        buf[2 * G][wave] = tot[0]; buf[2 * G + 1][wave] = tot[1];
    }
    __syncthreads();
    constexpr bool kRow = kWaves == 16;                 // a lane per wave, else every lane walks the waves in order
    const int at = kRow ? lane & 15 : 0;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        if constexpr (kRow) {
            const float mw = buf[g][at];
            m[g] = lane_value(row_reduce<true>(mw), 0);
            l[g] = lane_value(row_reduce<false>(mw > -INFINITY ? buf[G + g][at] * exp2_fast(mw - m[g]) : 0.f), 0);
        } else {
            float M = buf[g][0], L = 0.f;
#pragma unroll
            for (int w = 1; w < kWaves; ++w) M = fmaxf(M, buf[g][w]);
#pragma unroll
            for (int w = 0; w < kWaves; ++w) L += buf[g][w] > -INFINITY ? buf[G + g][w] * exp2_fast(buf[g][w] - M) : 0.f;
            m[g] = M; l[g] = L;
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if constexpr (kRow) tot[i] = lane_value(row_reduce<false>(buf[2 * G + i][at]), 0);
        else {
            float t = buf[2 * G + i][0];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) t += buf[2 * G + i][w];
            tot[i] = t;
        }
    }
}
// arg-min (kMin) or arg-max of (value, index) pairs, lowest index on ties; index < 0 = none
template <bool kMin>
__device__ __forceinline__ bool better(float v, int i, float bv, int bi)
{
    if (i < 0) return false;
    if (bi < 0) return true;
    if (kMin ? v < bv : v > bv) return true;
    return v == bv && i < bi;
}
template <bool kMin, int kCtrl>
__device__ __forceinline__ void arg_step(float& v, int& i)
{
    const float ov = dpp_f<kCtrl>(v);
    const int oi = dpp_i<kCtrl>(i);
    if (better<kMin>(ov, oi, v, i)) { v = ov; i = oi; }
}
template <bool kMin>
__device__ __forceinline__ void row_arg(float& v, int& i)
{
    arg_step<kMin, kDppXor1>(v, i);
    arg_step<kMin, kDppXor2>(v, i);
    arg_step<kMin, kDppHalfMirror>(v, i);
    arg_step<kMin, kDppMirror>(v, i);
}
// (`fbuf` and `ibuf` are the call's own: one barrier)
template <int kWaves, bool kMin>
__device__ __forceinline__ void block_arg(float& v, int& i, float* fbuf, int* ibuf)
{
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    row_arg<kMin>(v, i);
    {
        float bv = lane_value(v, 0);
        int bi = __builtin_amdgcn_readlane(i, 0);
#pragma unroll
        for (int r = 16; r < 64; r += 16) {
            const float ov = lane_value(v, r);
            const int oi = __builtin_amdgcn_readlane(i, r);
            if (better<kMin>(ov, oi, bv, bi)) { bv = ov; bi = oi; }
        }
        v = bv; i = bi;
    }
    if (lane == 0) { fbuf[wave] = v; ibuf[wave] = i; }
    __syncthreads();
    if constexpr (kWaves == 16) {
        v = fbuf[lane & 15]; i = ibuf[lane & 15];
        row_arg<kMin>(v, i);
        v = lane_value(v, 0); i = __builtin_amdgcn_readlane(i, 0);
    } else {
        v = fbuf[0]; i = ibuf[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w)
            if (better<kMin>(fbuf[w], ibuf[w], v, i)) { v = fbuf[w]; i = ibuf[w]; }
    }
}

// ------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(256) void decode_init_kernel(DecodeInitArgs a)
{
    const int n_imp = a.n_imp, E = a.n_imp + a.n_tbm, W = a.window, Nb = a.budget, N = a.seq_len;
    const int Tn = E + W;
    const int bkv = blockIdx.y;
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= Tn) return;

    int pos = -1, row = -1;
    float norm = 0.f;
    if (j < n_imp) {
        pos = a.kept_pos[(size_t)bkv * Nb + j];
        row = j;
        norm = a.k_norm[(size_t)bkv * E + j];
        a.st.row_norm[(size_t)bkv * Nb + j] = norm;
        a.st.entry_tok[(size_t)bkv * n_imp + j] = j;
        a.st.entry_count[(size_t)bkv * n_imp + j] = a.slot_count[(size_t)bkv * (n_imp + 1) + j];
    } else if (j < E) {
        const int i = j - n_imp;
        const int d = a.tbm_dest[(size_t)bkv * a.n_tbm + i];
        if (d >= 0 && d < n_imp) {
            pos = a.tbm_idx[(size_t)bkv * a.n_tbm + i];
            row = d;
            norm = a.k_norm[(size_t)bkv * E + j];
        }
    } else {
        row = n_imp + (j - E);
        pos = a.kept_pos[(size_t)bkv * Nb + row];
        const T* kr = reinterpret_cast<const T*>(a.st.k_cache) + ((size_t)bkv * (Nb + 1) + row) * D;
        float ss = 0.f;
        for (int d = 0; d < D; ++d) { const float x = to_float(kr[d]); ss = __builtin_fmaf(x, x, ss); }
        norm = sqrtf(ss);
        a.st.row_norm[(size_t)bkv * Nb + row] = norm;
    }
    const size_t o = (size_t)bkv * Tn + j;
    const bool live = row >= 0;
    const int cp = min(max(pos, 0), N - 1);
    a.st.tok_pos[o] = live ? pos : -1;
    a.st.tok_row[o] = row;
    a.st.tok_norm[o] = norm;
    a.st.tok_glo[o] = live ? a.s_glo[(size_t)bkv * N + cp] : 0.f;
    a.st.tok_past[o] = live ? a.s_loc[(size_t)bkv * N + cp] : 0.f;
    a.st.tok_cur[o] = 0.f;
    if (bkv == 0 && j == 0) *a.st.step_count = 0;
}

// ------------------------------------------------------------------------------------
// One block per (batch, kv-head) runs the whole step (kPart = 0, 256 threads, or 512 for longer tables: the step is a chain of short
// dependent phases, and every instruction a wave spends on a block-wide bookkeeping step is paid once
// per wave) while the cache is small.
//
// Large caches: one compute unit cannot pull the cache rows fast enough, nor walk the table, so the step is
// three or four launches in stream order.  Few heads, over slices of the token table:
//   decode_logits_kernel   slices of the table: every token's own row against the group's queries, logits to the
//                          workspace, the slice's maxima, sums and scalar totals to the record
//   decode_choose_kernel   the same slices and those of the centre rows, in one launch or two: weights, score update,
//                          window shift, the least important centre, centre cosines (phase 5)
//   decode_commit_kernel   one block per head: phases 6-7
// A token gathers its row although tokens share entries: the row comes from the L2, and the table then needs no
// second look at the rows' dots.  Many heads fill the chip without the table's slices, and the gathers then
// cost more than they save:
//   kPart = 1              slices of the cache rows: phase 1 (row dots, staged in the workspace)
//   kPart = 2              one block per head, 1024 threads: phases 2-4
//   kPart = 5              slices of the centre rows: phase 5
//   decode_commit_kernel   as above
// (us a step, table slices / row slices, head size 128, budget 2000: 8 heads of 4 q-heads 16.7 / 23.1, 32 heads
// 23.2 / 25.4; when the table's slices were four launches, 64 heads of 4 37.0 / 33.9, 256 heads of 4 86.4 / 66.9.)
// Nothing waits for another block inside a launch.  (Letting the last cosine block
// of a head run phases 6-7 itself saves a launch and was measured slower: the next launch's latency hides
// behind the sweep anyway.)
// What one launch leaves for the next lives in the workspace: the logits or the staged dots and row norms, and
// a hand-over record per head (kHand* offsets below).
// Dynamic LDS of the one-launch step and of kPart = 2 (floats): dot[G][budget] | rn[budget] | the entries' centre tokens
// [n_imp] when that fits, else the first two live in the caller's workspace (a.lds_floats == 0), the last where it is.
constexpr int kHandSelf = 0;       // [8]  new query . new key per q-head (log2 units)
constexpr int kHandNewNorm = 8;    //      norm of the new key
constexpr int kHandOldSc = 9;      // [4]  scalars of the token that left the window
constexpr int kHandOldPos = 13;    //      its position (int)
constexpr int kHandStar = 14;      //      the least important centre (int)
constexpr int kHandStep = 15;      //      tokens generated before this one (int)
constexpr int kHandPart = 20;      // [kDecodeMaxSlices][2] best cosine and its centre per row slice
constexpr int kHandStat = kHandPart + 2 * kDecodeMaxSlices;     // [18][kDecodeMaxSlices] per table slice: maxima [8], sums [8], totals of s_Glo and s_Loc
constexpr int kHandLeast = kHandStat + 18 * kDecodeMaxSlices;   // [2][kDecodeMaxSlices] least score and its centre (int) per table slice
constexpr int kHandOldRow = kHandLeast + 2 * kDecodeMaxSlices;  // key row, then value row, of the token that left the window

// table elements a pass of a table slice covers
constexpr int kTokTile = 128;
// What the logits launch leaves of a centre's own element, in pieces of 16 bytes ([piece][centre]): the group's logits, s_Glo,
// s_Loc^cur, s_Loc^past.
template <int G> constexpr int kCentrePieces = (G + 3 + 3) / 4;

// arg-min (kMin) or arg-max over the lanes of a wave, lowest index on ties; the same in every lane
template <bool kMin>
__device__ __forceinline__ void wave_arg(float& v, int& i)
{
    row_arg<kMin>(v, i);
    float bv = lane_value(v, 0);
    int bi = __builtin_amdgcn_readlane(i, 0);
#pragma unroll
    for (int r = 16; r < 64; r += 16) {
        const float ov = lane_value(v, r);
        const int oi = __builtin_amdgcn_readlane(i, r);
        if (better<kMin>(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
    v = bv; i = bi;
}

template <int D, int G>
__global__ __launch_bounds__(256) void decode_logits_kernel(DecodeStepArgs a)
{
    using T = bf16_t;
    constexpr int kLpr = Tile<T, D>::kChunksPerRow, kRows = 256 / kLpr;      // rows a block loads at a time
    constexpr int kAhead = kTokTile / kRows;
    static_assert(kAhead <= kLpr, "a lane per row");
    __shared__ float red[2 * G + 2][4];
    const int n_imp = a.n_imp, Tn = n_imp + a.n_tbm + a.window, Nb = a.budget;
    const int bkv = blockIdx.y, slice = blockIdx.x, tid = threadIdx.x;
    const int grp = tid / kLpr, piece = tid % kLpr;
    const char* Kc = reinterpret_cast<const char*>(a.st.k_cache) + (size_t)bkv * (Nb + 1) * D * sizeof(T);
    const float* row_norm = a.st.row_norm + (size_t)bkv * Nb;
    const int32_t* tok_row = a.st.tok_row + (size_t)bkv * Tn;
    const size_t tok0 = (size_t)bkv * Tn;
    const char* qn = reinterpret_cast<const char*>(a.q_new) + (size_t)bkv * G * D * sizeof(T);
    const char* kn = reinterpret_cast<const char*>(a.k_new) + (size_t)bkv * D * sizeof(T);
    float* logits = a.ws + (size_t)bkv * G * Tn;
    f32x4_t* centres = reinterpret_cast<f32x4_t*>(a.ws + a.centre_at) + (size_t)bkv * kCentrePieces<G> * n_imp;
    const int32_t* entry_tok = a.st.entry_tok + (size_t)bkv * n_imp;
    float* hand = a.hand + (size_t)bkv * kDecodeHandFloats;

    frag_t qp[G];
#pragma unroll
    for (int g = 0; g < G; ++g) qp[g] = *reinterpret_cast<const frag_t*>(qn + ((size_t)g * kLpr + piece) * 16);

    float m[G], l[G], tot[2] = {0.f, 0.f};                   // this thread's table elements
#pragma unroll
    for (int g = 0; g < G; ++g) { m[g] = -INFINITY; l[g] = 0.f; }
    const int t_end = min((slice + 1) * a.tok_slice, Tn);
    for (int j0 = slice * a.tok_slice; j0 < t_end; j0 += kTokTile) {
        int rr[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) { const int j = j0 + u * kRows + grp; rr[u] = j < t_end ? tok_row[j] : -1; }
        const int j = j0 + piece * kRows + grp;              // of the rows a lane group loads, lane i takes on the i-th one's token
        const bool mine = piece < kAhead && j < t_end;
        const int r = mine ? tok_row[j] : -1;
        const float tn = mine ? a.st.tok_norm[tok0 + j] : 0.f, tg = mine ? a.st.tok_glo[tok0 + j] : 0.f;
        const float tp = mine ? a.st.tok_past[tok0 + j] : 0.f, tc = mine ? a.st.tok_cur[tok0 + j] : 0.f;
        frag_t fk[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) fk[u] = load_frag_or_zero(Kc, ((size_t)max(rr[u], 0) * kLpr + piece) * 16, rr[u] >= 0);
        const float rn = r >= 0 ? row_norm[r] : 0.f;
        const bool centre = r >= 0 && r < n_imp && entry_tok[r] == j;
        float dot[G];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float d = group_sum<kLpr>(dot8_bf16(fk[u], qp[g]));
                dot[g] = u == 0 || piece == u ? d : dot[g];
            }
        if (r >= 0) {
            const float c = a.scale_log2e * (rn > 0.f ? tn / rn : 0.f);
            f32x4_t left[kCentrePieces<G>];
            left[kCentrePieces<G> - 1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float x = c * dot[g];
                left[g / 4][g % 4] = x;
                const float m_new = fmaxf(m[g], x), ref = m_new > -INFINITY ? m_new : 0.f;
                l[g] = l[g] * exp2_fast(m[g] - ref) + exp2_fast(x - ref);
                m[g] = m_new;
                logits[(size_t)g * Tn + j] = x;
            }
            tot[0] += tg;
            tot[1] += tp + tc;
            left[G / 4][G % 4] = tg; left[(G + 1) / 4][(G + 1) % 4] = tc; left[(G + 2) / 4][(G + 2) % 4] = tp;
            if (centre) {
#pragma unroll
                for (int i = 0; i < kCentrePieces<G>; ++i) centres[(size_t)i * n_imp + r] = left[i];
            }
        }
    }
    // the slice's maxima, sums relative to them, and totals
    block_softmax<4, G>(m, l, tot, red);
    if (tid == 0) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            hand[kHandStat + g * kDecodeMaxSlices + slice] = m[g];
            hand[kHandStat + (8 + g) * kDecodeMaxSlices + slice] = l[g];
        }
        hand[kHandStat + 16 * kDecodeMaxSlices + slice] = tot[0];
        hand[kHandStat + 17 * kDecodeMaxSlices + slice] = tot[1];
    }
    if (slice == 0 && tid < kLpr) {                          // the new token
        const frag_t new_k = *reinterpret_cast<const frag_t*>(kn + piece * 16);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float d = group_sum<kLpr>(dot8_bf16(new_k, qp[g]));
            if (piece == 0) hand[kHandSelf + g] = a.scale_log2e * d;
        }
        const float ss = group_sum<kLpr>(frag_sumsq<T>(new_k));
        if (piece == 0) {
            hand[kHandNewNorm] = sqrtf(ss);
            reinterpret_cast<int*>(hand)[kHandStep] = a.step >= 0 ? a.step : *a.st.step_count;
        }
    }
}

// Weights, the least important centre and its cosines.
//   kChoose              in one launch: every block forms the scores of all centres for itself, from what the launch before left
//                        of them (the table's scalars are being updated by the other blocks)
//   kWeights, kCosines   in two: the weights and each table slice's least important centre; the least of all and its cosines
enum ChooseStep { kChoose, kWeights, kCosines };
template <int D, int G, int kBlock, ChooseStep kStep>
__global__ __launch_bounds__(kBlock) void decode_choose_kernel(DecodeStepArgs a)
{
    using T = bf16_t;
    constexpr bool kDoWeights = kStep != kCosines, kDoCosines = kStep != kWeights;
    constexpr int kWaves = kBlock / kWave;
    constexpr int kLpr = Tile<T, D>::kChunksPerRow, kRows = kBlock / kLpr;     // rows a block loads at a time
    constexpr int kAhead = kTokTile / kRows;                 // row loads in flight per thread
    constexpr int kCen = 4, kPieces = kCentrePieces<G>;      // centres in flight per thread
    __shared__ float fbuf[2][kWaves];
    __shared__ int ibuf[2][kWaves];
    const int n_imp = a.n_imp, E = a.n_imp + a.n_tbm, Tn = E + a.window, Nb = a.budget;
    const int bkv = blockIdx.y, slice = blockIdx.x, tid = threadIdx.x, lane = tid % kWave;
    const int grp = tid / kLpr, piece = tid % kLpr;
    const size_t tok0 = (size_t)bkv * Tn;
    char* Kc = reinterpret_cast<char*>(a.st.k_cache) + (size_t)bkv * (Nb + 1) * D * sizeof(T);
    char* Vc = reinterpret_cast<char*>(a.st.v_cache) + (size_t)bkv * (Nb + 1) * D * sizeof(T);
    float* hand = a.hand + (size_t)bkv * kDecodeHandFloats;
    int* hand_i = reinterpret_cast<int*>(hand);

    // ---- what waits for nothing: the first centres' scalars, the slices' records, the first centre rows
    f32x4_t cen[kCen][kPieces];
    auto load_scalars = [&](int r0) __attribute__((always_inline)) {
        const f32x4_t* centres = reinterpret_cast<const f32x4_t*>(a.ws + a.centre_at) + (size_t)bkv * kPieces * n_imp;
#pragma unroll
        for (int u = 0; u < kCen; ++u)
#pragma unroll
            for (int i = 0; i < kPieces; ++i) cen[u][i] = centres[(size_t)i * n_imp + min(r0 + u * kBlock, n_imp - 1)];
    };
    if constexpr (kStep == kChoose) load_scalars(tid);
    // (every wave combines the records for itself: a row of 16 lanes per q-head, two slices a lane)
    static_assert(kDecodeMaxSlices == 32, "two slices a lane");
    constexpr int kPasses = (G + 3) / 4;
    const int row = lane / 16, at = lane % 16;
    float sm[kPasses][2], sl[kPasses][2], self[kPasses], st[2];
    if constexpr (kDoWeights) {
        auto record = [&](int what, bool there, float none, float (&v)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 2; ++i) v[i] = there && at + 16 * i < a.n_tok_slices ? hand[kHandStat + what * kDecodeMaxSlices + at + 16 * i] : none;
        };
#pragma unroll
        for (int q = 0; q < kPasses; ++q) {
            const int g = 4 * q + row;
            record(g, g < G, -INFINITY, sm[q]);
            record(8 + g, g < G, 0.f, sl[q]);
            self[q] = g < G ? hand[kHandSelf + g] : 0.f;
        }
        record(16 + row, row < 2, 0.f, st);
    }
    const int c_lo = slice * a.slice_rows, c_end = min(c_lo + a.slice_rows, n_imp);       // this block's centre rows: none where c_lo >= n_imp
    frag_t rows[kAhead];
    auto load_centres = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            rows[u] = load_frag_or_zero(Kc, ((size_t)(s0 + u * kRows + grp) * kLpr + piece) * 16, s0 + u * kRows + grp < c_end);
    };
    if constexpr (kDoCosines) load_centres(c_lo);

    float bv = 0.f;                                          // the least important centre seen
    int bi = -1, s_star = 0;
    frag_t sp = zero_frag();                                 // its key
    auto star_row = [&]() __attribute__((always_inline)) {
        s_star = max(bi, 0);
        sp = *reinterpret_cast<const frag_t*>(Kc + ((size_t)s_star * kLpr + piece) * 16);
    };
    if constexpr (kDoWeights) {
        float m[G], inv[G], self_w[G], self_tot = 0.f;
#pragma unroll
        for (int q = 0; q < kPasses; ++q) {
            const float top = fmaxf(row_reduce<true>(fmaxf(sm[q][0], sm[q][1])), self[q]);
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < 2; ++i) sum += sm[q][i] > -INFINITY ? sl[q][i] * exp2_fast(sm[q][i] - top) : 0.f;
            const float own = exp2_fast(self[q] - top), over = 1.0f / (row_reduce<false>(sum) + own);
#pragma unroll
            for (int g = 4 * q; g < min(G, 4 * q + 4); ++g) {
                m[g] = lane_value(top, 16 * (g - 4 * q));
                inv[g] = lane_value(over, 16 * (g - 4 * q));
                self_w[g] = lane_value(own * over, 16 * (g - 4 * q));
                self_tot += self_w[g];
            }
        }
        // Eq. 2 factor on the updated scalars: this step adds one unit of weight per q-head to both totals
        const float both = row_reduce<false>(st[0] + st[1]);
        const float s_glo = lane_value(both, 0) + (float)G, s_loc = lane_value(both, 16) + (float)G;
        const float align = s_glo > 0.f ? s_loc / s_glo : 0.f;
        auto weights = [&](const float (&x)[G], float (&w)[G]) __attribute__((always_inline)) {
            float add = 0.f;
#pragma unroll
            for (int g = 0; g < G; ++g) { w[g] = exp2_fast(x[g] - m[g]) * inv[g]; add += w[g]; }
            return add;
        };
        if constexpr (kStep == kChoose) {
            for (int r0 = tid;;) {
#pragma unroll
                for (int u = 0; u < kCen; ++u) {
                    const int r = r0 + u * kBlock;
                    float x[G], w[G];
#pragma unroll
                    for (int g = 0; g < G; ++g) x[g] = cen[u][g / 4][g % 4];
                    const float tg = cen[u][G / 4][G % 4], tc = cen[u][(G + 1) / 4][(G + 1) % 4], tp = cen[u][(G + 2) / 4][(G + 2) % 4];
                    const float add = weights(x, w), sc = fmaxf((tg + add) * align, tp + (tc + add));
                    if (r < n_imp && better<true>(sc, r, bv, bi)) { bv = sc; bi = r; }
                }
                r0 += kCen * kBlock;
                if (r0 - tid >= n_imp) break;                // block-uniform
                load_scalars(r0);
            }
            block_arg<kWaves, true>(bv, bi, fbuf[0], ibuf[0]);
            star_row();
        }

        // ---- the block's table elements; the oldest window token leaves, the new one takes its place
        const float* logits = a.ws + (size_t)bkv * G * Tn;
        const int32_t* entry_tok = a.st.entry_tok + (size_t)bkv * n_imp;
        const int step = hand_i[kHandStep], ring = step % a.window, jo = E + ring, ro = n_imp + ring;
        const int t_end = min((slice + 1) * a.tok_slice, Tn);
        for (int j = slice * a.tok_slice + tid; j < t_end; j += kBlock) {
            const int r = a.st.tok_row[tok0 + j];
            float w[G];
#pragma unroll
            for (int g = 0; g < G; ++g) w[g] = 0.f;
            if (r >= 0) {
                float x[G];
#pragma unroll
                for (int g = 0; g < G; ++g) x[g] = logits[(size_t)g * Tn + j];
                const float add = weights(x, w), past = a.st.tok_past[tok0 + j];
                const float glo = a.st.tok_glo[tok0 + j] + add, cur = a.st.tok_cur[tok0 + j] + add;
                a.st.tok_glo[tok0 + j] = glo;
                a.st.tok_cur[tok0 + j] = cur;
                if (kStep == kWeights && r < n_imp && entry_tok[r] == j) {       // a class centre's own element
                    const float sc = fmaxf(glo * align, past + cur);
                    if (better<true>(sc, r, bv, bi)) { bv = sc; bi = r; }
                }
                if (j == jo) { hand[kHandOldSc + 1] = glo; hand[kHandOldSc + 2] = past; hand[kHandOldSc + 3] = cur; }
            }
            if (j == jo) {
                const float norm = hand[kHandNewNorm];
                hand[kHandOldSc] = a.st.tok_norm[tok0 + j];
                hand_i[kHandOldPos] = a.st.tok_pos[tok0 + j];
                a.st.tok_pos[tok0 + j] = a.seq_len + step; a.st.tok_row[tok0 + j] = ro; a.st.tok_norm[tok0 + j] = norm;
                a.st.tok_glo[tok0 + j] = self_tot; a.st.tok_past[tok0 + j] = 0.f; a.st.tok_cur[tok0 + j] = self_tot;
                a.st.row_norm[(size_t)bkv * Nb + ro] = norm;
            }
            if (a.attn_opt) {
#pragma unroll
                for (int g = 0; g < G; ++g) a.attn_opt[((size_t)bkv * G + g) * (Tn + 1) + j] = w[g];
            }
        }
        if constexpr (kStep == kWeights) {
            block_arg<kWaves, true>(bv, bi, fbuf[0], ibuf[0]);
            if (tid == 0) { hand[kHandLeast + slice] = bv; hand_i[kHandLeast + kDecodeMaxSlices + slice] = bi; }
        }
        if (slice == 0) {
            if (grp == 0) {
                frag_t* const hand_row = reinterpret_cast<frag_t*>(hand + kHandOldRow);
                char* const k_at = Kc + ((size_t)ro * kLpr + piece) * 16;
                char* const v_at = Vc + ((size_t)ro * kLpr + piece) * 16;
                hand_row[piece] = *reinterpret_cast<const frag_t*>(k_at);
                hand_row[kLpr + piece] = *reinterpret_cast<const frag_t*>(v_at);
                const size_t new_at = ((size_t)bkv * kLpr + piece) * 16;
                *reinterpret_cast<frag_t*>(k_at) = *reinterpret_cast<const frag_t*>(reinterpret_cast<const char*>(a.k_new) + new_at);
                *reinterpret_cast<frag_t*>(v_at) = *reinterpret_cast<const frag_t*>(reinterpret_cast<const char*>(a.v_new) + new_at);
            }
            if (a.attn_opt && tid == 0) {
#pragma unroll
                for (int g = 0; g < G; ++g) a.attn_opt[((size_t)bkv * G + g) * (Tn + 1) + Tn] = self_w[g];
            }
        }
    } else {
        bv = lane < a.n_tok_slices ? hand[kHandLeast + lane] : 0.f;
        bi = lane < a.n_tok_slices ? hand_i[kHandLeast + kDecodeMaxSlices + lane] : -1;
        wave_arg<true>(bv, bi);
        star_row();
    }
    if constexpr (kDoCosines) {
        if (slice == 0 && tid == 0) hand_i[kHandStar] = s_star;
        if (c_lo >= n_imp) return;                           // block-uniform
        // ---- its cosines with the block's centre rows (as phase 5 of the step kernel)
        float cv = 0.f;
        int ci = -1;
        const float rn_star = row_inv_norm<T>(group_sum<kLpr>(frag_sumsq<T>(sp)));
        for (int s0 = c_lo; s0 < c_end; s0 += kTokTile) {
            if (s0 != c_lo) load_centres(s0);
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int s = s0 + u * kRows + grp;
                if (s >= c_end) break;                       // uniform over the row's lanes
                const float d = group_sum<kLpr>(frag_dot<T>(rows[u], sp));
                const float e2 = group_sum<kLpr>(frag_sumsq<T>(rows[u]));
                const float sim = (d * row_inv_norm<T>(e2)) * rn_star;
                if (piece == 0 && s != s_star && better<false>(sim, s, cv, ci)) { cv = sim; ci = s; }
            }
        }
        block_arg<kWaves, false>(cv, ci, fbuf[1], ibuf[1]);
        if (tid == 0) { hand[kHandPart + 2 * slice] = cv; hand_i[kHandPart + 2 * slice + 1] = ci; }
    }
}

// Merge at class-centre level: the row piece at `to` becomes the mean of entry b's (there) and entry a's, weighted by their counts;
// keys as unit vectors, scaled to b's norm.  (A value counts as a vector of norm 1.)
template <typename T>
__device__ __forceinline__ void merge_rows(char* to, const frag_t& from, bool key, float ca, float cb, float na, float nb)
{
    using P = Pack<T>;
    constexpr int kE = P::kElems;
    const float ra = !key ? 1.f : na > 0.f ? 1.0f / na : 0.f, rb = !key ? 1.f : nb > 0.f ? 1.0f / nb : 0.f;
    const float scale = key ? nb : 1.f;
    float xa[kE], xb[kE];
    P::unpack(from, xa);
    P::unpack(*reinterpret_cast<const frag_t*>(to), xb);
#pragma unroll
    for (int i = 0; i < kE; ++i) xb[i] = scale * ((cb * (xb[i] * rb) + ca * (xa[i] * ra)) / (ca + cb));
    *reinterpret_cast<frag_t*>(to) = P::pack(xb);
}

// The last launch of the sliced step, one block per head: merge at class-centre level or evict, followers follow (as phases 6
// and 7 of the step kernel).  Bound by two dependent round trips: what the launches before left and the table's rows, then
// the chosen entries' rows.  Every wave finds the winner for itself, and the lanes that read a row, count or norm are those that write it,
// so that no barrier is needed.
constexpr int kCommitBlock = 512;
template <typename T, int D>
__global__ __launch_bounds__(kCommitBlock) void decode_commit_kernel(DecodeStepArgs a)
{
    constexpr int kLpr = Tile<T, D>::kChunksPerRow;
    constexpr int kUnroll = 8;                               // table elements in flight per thread
    const int n_imp = a.n_imp, E = n_imp + a.n_tbm, W = a.window, Tn = E + W, Nb = a.budget;
    const int bkv = blockIdx.x, tid = threadIdx.x, lane = tid % kWave;
    const int piece = tid % kLpr;
    const bool row_lane = tid < 2 * kLpr, key = tid < kLpr;  // a piece of a key, or of the value
    static_assert(2 * kLpr <= kWave, "both rows in one wave");
    char* Kc = reinterpret_cast<char*>(a.st.k_cache) + (size_t)bkv * (Nb + 1) * D * sizeof(T);
    char* Vc = reinterpret_cast<char*>(a.st.v_cache) + (size_t)bkv * (Nb + 1) * D * sizeof(T);
    float* row_norm = a.st.row_norm + (size_t)bkv * Nb;
    int32_t* entry_count = a.st.entry_count + (size_t)bkv * n_imp;
    int32_t* tok_pos = a.st.tok_pos + (size_t)bkv * Tn;
    int32_t* tok_row = a.st.tok_row + (size_t)bkv * Tn;
    float* tok_norm = a.st.tok_norm + (size_t)bkv * Tn;
    float* tok_glo = a.st.tok_glo + (size_t)bkv * Tn;
    float* tok_past = a.st.tok_past + (size_t)bkv * Tn;
    float* tok_cur = a.st.tok_cur + (size_t)bkv * Tn;
    const float* hand = a.hand + (size_t)bkv * kDecodeHandFloats;
    const int* hand_i = reinterpret_cast<const int*>(hand);
    const frag_t* hand_row = reinterpret_cast<const frag_t*>(hand + kHandOldRow);

    const int s_star = hand_i[kHandStar], step = hand_i[kHandStep];
    static_assert(kDecodeMaxSlices <= kWave, "a slice per lane");
    float cv = lane < a.n_slices ? hand[kHandPart + 2 * lane] : 0.f;
    int ci = lane < a.n_slices ? hand_i[kHandPart + 2 * lane + 1] : -1;
    int rr[kUnroll];
    auto load_rows_of = [&](int j0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) rr[u] = j0 + u * kCommitBlock < E ? tok_row[j0 + u * kCommitBlock] : -1;
    };
    load_rows_of(tid);
    const frag_t old_row = row_lane ? hand_row[tid] : zero_frag();               // the token that left the window
    const float old_norm = hand[kHandOldSc], old_glo = hand[kHandOldSc + 1], old_past = hand[kHandOldSc + 2], old_cur = hand[kHandOldSc + 3];
    const int old_pos = hand_i[kHandOldPos];

    wave_arg<false>(cv, ci);                                 // the slices' winners, lowest centre on ties
    const bool merged = ci >= 0 && cv > a.tau;
    const int dst = merged ? ci : -1;
    const int f = a.st.entry_tok[(size_t)bkv * n_imp + s_star];
    if (row_lane) {
        char* const X = key ? Kc : Vc;
        char* const star = X + ((size_t)s_star * kLpr + piece) * 16;
        if (merged) {
            char* const to = X + ((size_t)dst * kLpr + piece) * 16;
            const int na_count = entry_count[s_star], nb_count = entry_count[dst];
            merge_rows<T>(to, *reinterpret_cast<const frag_t*>(star), key, (float)na_count, (float)nb_count, row_norm[s_star], row_norm[dst]);
            if (tid == 0) entry_count[dst] = nb_count + na_count;
        }
        // the token that left the window is the new centre of entry s_star and takes the departed centre's table element
        *reinterpret_cast<frag_t*>(star) = old_row;
    }
    if (tid == 0) {
        entry_count[s_star] = 1;
        row_norm[s_star] = old_norm;
        tok_pos[f] = old_pos; tok_row[f] = s_star; tok_norm[f] = old_norm;
        tok_glo[f] = old_glo; tok_past[f] = old_past; tok_cur[f] = old_cur;
        if (a.decision_opt) { a.decision_opt[(size_t)bkv * 2] = s_star; a.decision_opt[(size_t)bkv * 2 + 1] = dst; }
        if (a.sim_opt) a.sim_opt[bkv] = ci >= 0 ? cv : -INFINITY;
        if (bkv == 0) *a.st.step_count = step + 1;           // (every block reads the hand-over copy)
    }
    for (int j0 = tid; j0 < E; j0 += kCommitBlock * kUnroll) {
        if (j0 != tid) load_rows_of(j0);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int j = j0 + u * kCommitBlock;
            if (rr[u] != s_star || j == f) continue;
            if (merged) {
                tok_row[j] = dst;
            } else {
                tok_row[j] = -1; tok_pos[j] = -1;
                tok_norm[j] = 0.f; tok_glo[j] = 0.f; tok_past[j] = 0.f; tok_cur[j] = 0.f;
            }
        }
    }
    // a full window of queries: s_Loc^cur becomes s_Loc^past (Sec. 3.3)
    if ((step + 1) % W == 0) {                               // block-uniform
        __syncthreads();
        for (int j = tid; j < Tn; j += kCommitBlock) { tok_past[j] = tok_cur[j]; tok_cur[j] = 0.f; }
    }
}

template <typename T, int D, int G, int kBlock, int kPart>
__global__ __launch_bounds__(kBlock) void decode_step_kernel(DecodeStepArgs a)
{
    constexpr bool kAll = kPart == 0;
    constexpr bool kDoDots = kAll || kPart == 1, kDoSoftmax = kAll || kPart == 2;
    constexpr bool kDoCos = kAll || kPart == 5;
    static_assert(kAll || kPart == 1 || kPart == 2 || kPart == 5, "parts");
    static_assert(kHandOldRow % 4 == 0 && kHandOldRow + 2 * D * (int)sizeof(T) / 4 <= kDecodeHandFloats, "hand-over record");
    constexpr int kWaves = kBlock / kWave;
    constexpr int kLpr = Tile<T, D>::kChunksPerRow;          // lanes per cache row
    constexpr int kUnroll = 4;                               // independent loads in flight per thread

    extern __shared__ float dyn_lds[];
    __shared__ float fbuf[2][kWaves];
    __shared__ int ibuf[2][kWaves];
    __shared__ float vbuf[2 * G + 2][kWaves];                // the softmax's reduction
    __shared__ frag_t star_k[kLpr];                          // the least important centre's key
    __shared__ float old_sc[4];                              // of the token that leaves the window: norm, glo, past, cur
    __shared__ float sh_newnorm;

    const int n_imp = a.n_imp, E = a.n_imp + a.n_tbm, W = a.window, Nb = a.budget;
    const int Tn = E + W;
    const int bkv = blockIdx.y, slice = blockIdx.x;          // slice = 0 unless the part sweeps rows
    const int tid = threadIdx.x;
    // tokens generated before this one: the caller's count, or the counter kept in the state.  The
    // counter is advanced after every block has read it: by a separate launch after the one-launch
    // step (by the step itself when nobody reads it); in the sliced step the first part copies it into
    // every head's hand-over record, the later parts read that copy, and the last part advances it.
    const int step = a.step >= 0 ? a.step
                   : (kPart >= 2 ? reinterpret_cast<const int*>(a.hand + (size_t)bkv * kDecodeHandFloats)[kHandStep] : *a.st.step_count);
    const int lane = tid % kWave, wave = tid / kWave;
    const int grp = tid / kLpr, piece = tid % kLpr;

    char* Kc = reinterpret_cast<char*>(a.st.k_cache) + (size_t)bkv * (Nb + 1) * D * sizeof(T);
    char* Vc = reinterpret_cast<char*>(a.st.v_cache) + (size_t)bkv * (Nb + 1) * D * sizeof(T);
    float* row_norm = a.st.row_norm + (size_t)bkv * Nb;
    int32_t* entry_count = a.st.entry_count + (size_t)bkv * n_imp;
    int32_t* entry_tok = a.st.entry_tok + (size_t)bkv * n_imp;
    int32_t* tok_pos = a.st.tok_pos + (size_t)bkv * Tn;
    int32_t* tok_row = a.st.tok_row + (size_t)bkv * Tn;
    float* tok_norm = a.st.tok_norm + (size_t)bkv * Tn;
    float* tok_glo = a.st.tok_glo + (size_t)bkv * Tn;
    float* tok_past = a.st.tok_past + (size_t)bkv * Tn;
    float* tok_cur = a.st.tok_cur + (size_t)bkv * Tn;
    // kPart = 1 writes the staged arrays to the workspace; kPart = 2 copies them into LDS first when they fit
    float* ws_stage = a.ws + (size_t)bkv * ((size_t)(G + 1) * Nb);
    const bool in_lds = a.lds_floats > 0 && (kAll || kPart == 2);   // block-uniform
    float* stage = in_lds ? dyn_lds : ws_stage;
    float* hand = kAll ? nullptr : a.hand + (size_t)bkv * kDecodeHandFloats;
    int* hand_i = reinterpret_cast<int*>(hand);
    frag_t* hand_row = reinterpret_cast<frag_t*>(hand + kHandOldRow);
    // rows of this block's sweeps: every row, or the block's slice
    const int r_lo = kAll ? 0 : slice * a.slice_rows;
    const int r_end = kAll ? Nb : min(r_lo + a.slice_rows, Nb + 1);           // phase 1 (row Nb = the new key)
    const int c_end = kAll ? n_imp : min(r_lo + a.slice_rows, n_imp);        // phase 5
    float* dot = stage;                                      // [G][budget] q_g . cache row
    float* rn_of = stage + (size_t)G * Nb;                   // [budget] copy of row_norm
    const char* qn = reinterpret_cast<const char*>(a.q_new) + (size_t)bkv * G * D * sizeof(T);
    const char* kn = reinterpret_cast<const char*>(a.k_new) + (size_t)bkv * D * sizeof(T);
    const char* vn = reinterpret_cast<const char*>(a.v_new) + (size_t)bkv * D * sizeof(T);

    // ---- phase 1: q_g . (every cache row), the new token's own key included as row Nb ----
    // A row is kLpr consecutive lanes x 16 bytes, so a wave-wide load covers 64 / kLpr
    // whole rows (fully coalesced); each lane forms the partial dots of its elements (16 bits: with
    // v_dot2) and the kLpr partials are added with DPP.  One dot per cache ROW serves every
    // token that shares the entry.
    // Everything this thread will need from global memory that does not depend on earlier
    // phases is requested here, behind the first row loads, so that the round trips overlap:
    // the first batch of table elements (all of them for small tables), the centre token of
    // "its" entry, its share of the row norms, the new token's row.
    constexpr int kRowsPerWave = kWave / kLpr;               // whole rows per wave-wide load
    constexpr int kRowsPerPass = kWaves * kRowsPerWave;
    constexpr int kInFlight = kAll ? 2048 / kBlock : 4;                  // row loads in flight per lane
    const int sub = lane / kLpr;                             // this lane's row within the wave's load
    const int mine = wave * kRowsPerWave + sub;              // and within the block's
    frag_t row_pre[kInFlight];                               // the first batch of rows: phase 1's, and in the one-launch step phase 5's
    frag_t new_k = zero_frag(), new_v = zero_frag();
    float m[G], inv[G], self[G];                             // (self: new query . new key, in log2 units)
    float tot2[2] = {0.f, 0.f};                              // sum of s_Glo, sum of s_Loc
    float self_tot = 0.f;
    int s_star = 0, f = 0;
    float cv = 0.f;
    int ci = -1;
    int pre_rr[kUnroll];
    float pre_tn[kUnroll], pre_tg[kUnroll], pre_tp[kUnroll], pre_tc[kUnroll];
    // the entries' centre tokens, in LDS behind the staged arrays where these are there
    const bool ct_in_lds = in_lds && a.lds_centres > 0;      // block-uniform
    int* sh_ct = reinterpret_cast<int*>(dyn_lds) + (size_t)(G + 1) * Nb;
    constexpr int kCt = 2;                                   // looked up ahead per thread
    int pre_ct[kCt];
    auto preload_centres = [&]() {
#pragma unroll
        for (int u = 0; u < kCt; ++u) pre_ct[u] = tid + u * kBlock < n_imp ? entry_tok[tid + u * kBlock] : -1;
    };
    auto store_centres = [&]() {
        if (!ct_in_lds) return;                              // block-uniform
#pragma unroll
        for (int u = 0; u < kCt; ++u)
            if (tid + u * kBlock < n_imp) sh_ct[tid + u * kBlock] = pre_ct[u];
        for (int i = tid + kCt * kBlock; i < n_imp; i += kBlock) sh_ct[i] = entry_tok[i];
    };
    auto centre_of = [&](int r) __attribute__((always_inline)) { return r < 0 || r >= n_imp ? -1 : ct_in_lds ? sh_ct[r] : entry_tok[r]; };
    auto preload_table = [&]() {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (u * kBlock >= Tn) break;                     // block-uniform, as in the sweeps: a batch ends where the table does
            const int j = tid + u * kBlock;
            const bool ok = j < Tn;
            pre_rr[u] = ok ? tok_row[j] : -1;
            pre_tn[u] = ok ? tok_norm[j] : 0.f;
            pre_tg[u] = ok ? tok_glo[j] : 0.f;
            pre_tp[u] = ok ? tok_past[j] : 0.f;
            pre_tc[u] = ok ? tok_cur[j] : 0.f;
        }
    };
    // the token that leaves the window: its rows and position (its scalars come from the thread that updates them)
    const int ring = step % W;
    const int jo = E + ring, ro = n_imp + ring;
    const bool row_lane = grp < 2;                           // a piece of a key, or of the value beside it
    static_assert(2 * kLpr <= kWave, "both rows in one wave");
    char* const X = grp == 0 ? Kc : Vc;
    frag_t pre_old = zero_frag();
    int pre_old_pos = 0;
    auto preload_old = [&]() {
        if (row_lane) pre_old = *reinterpret_cast<const frag_t*>(X + ((size_t)ro * kLpr + piece) * 16);
        if (tid == 0) pre_old_pos = tok_pos[jo];
    };
    if constexpr (kDoDots) {
        frag_t qp[G];
#pragma unroll
        for (int g = 0; g < G; ++g) qp[g] = *reinterpret_cast<const frag_t*>(qn + ((size_t)g * kLpr + piece) * 16);
        new_k = *reinterpret_cast<const frag_t*>(kn + piece * 16);
        auto load_rows = [&](int base, frag_t (&fk)[kInFlight]) __attribute__((always_inline)) {
            const int r0 = base + mine;
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                const int r = r0 + u * kRowsPerPass;
                if (kAll && base + u * kRowsPerPass >= r_end) break;                 // block-uniform
                fk[u] = r < Nb ? *reinterpret_cast<const frag_t*>(Kc + ((size_t)r * kLpr + piece) * 16) : new_k;
            }
        };
        load_rows(r_lo, row_pre);
        if constexpr (kAll) preload_table();
        const float rn_mine = (kAll && tid < Nb) ? row_norm[tid] : 0.f;
        if (grp == 1) new_v = *reinterpret_cast<const frag_t*>(vn + piece * 16);
        if constexpr (kAll) { preload_old(); preload_centres(); }
        auto dots = [&](int base, const frag_t (&fk)[kInFlight]) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                const int r = base + mine + u * kRowsPerPass;
                if (kAll && base + u * kRowsPerPass >= r_end) break;                 // block-uniform
                if (r >= r_end) break;                       // uniform over the row's lanes
                float d[G];
#pragma unroll
                for (int g = 0; g < G; ++g) d[g] = group_sum<kLpr>(frag_dot<T>(fk[u], qp[g]));
                if (piece == 0) {
                    if (kAll || r < Nb) {
#pragma unroll
                        for (int g = 0; g < G; ++g) dot[(size_t)g * Nb + r] = d[g];
                    } else {
#pragma unroll
                        for (int g = 0; g < G; ++g) {
                            hand[kHandSelf + g] = a.scale_log2e * d[g];
                        }
                    }
                }
            }
        };
        dots(r_lo, row_pre);
        for (int base = r_lo + kRowsPerPass * kInFlight; base < r_end; base += kRowsPerPass * kInFlight) {
            frag_t fk[kInFlight];
            load_rows(base, fk);
            dots(base, fk);
        }
        if constexpr (kAll) {                                // the new token's, by every wave
#pragma unroll
            for (int g = 0; g < G; ++g) self[g] = a.scale_log2e * group_sum<kLpr>(frag_dot<T>(new_k, qp[g]));
        }
        if constexpr (kAll) store_centres();
        for (int r = r_lo + tid; r < min(r_end, Nb); r += kBlock) rn_of[r] = (kAll && r == tid) ? rn_mine : row_norm[r];
        if (grp == 0 && (kAll || slice == 0)) {
            const float ss = group_sum<kLpr>(frag_sumsq<T>(new_k));
            if (piece == 0) { sh_newnorm = sqrtf(ss); if (!kAll) hand[kHandNewNorm] = sqrtf(ss); }
        }
    }   // kDoDots
    if constexpr (kPart == 1) {
        if (slice == 0 && tid == 0) hand_i[kHandStep] = step;
        return;
    }
    if constexpr (kPart == 2) {
        // what the dots launch left: the new token's own logits and norm, the staged arrays
        preload_table();
        preload_old();
        preload_centres();
#pragma unroll
        for (int g = 0; g < G; ++g) self[g] = hand[kHandSelf + g];
        if (tid == 0) sh_newnorm = hand[kHandNewNorm];
        if (grp == 0) new_k = *reinterpret_cast<const frag_t*>(kn + piece * 16);
        if (grp == 1) new_v = *reinterpret_cast<const frag_t*>(vn + piece * 16);
        if (in_lds) {
            constexpr int kCopy = 8;                         // loads in flight per thread
            for (int i0 = tid; i0 < (G + 1) * Nb; i0 += kBlock * kCopy) {
                float t[kCopy];
#pragma unroll
                for (int u = 0; u < kCopy; ++u) t[u] = i0 + u * kBlock < (G + 1) * Nb ? ws_stage[i0 + u * kBlock] : 0.f;
#pragma unroll
                for (int u = 0; u < kCopy; ++u)
                    if (i0 + u * kBlock < (G + 1) * Nb) dyn_lds[i0 + u * kBlock] = t[u];
            }
        }
        store_centres();
    }
    if constexpr (kDoSoftmax) {
    __syncthreads();

    // ---- phase 2: softmax over the live tokens and the new token (Eq. 1) ---------------
    // logit of token j in row r: scale * (|k_j| / |centre of r|) * (q . row r).  Two sweeps over the table: logits with their
    // maxima, sums relative to these and the scalars' totals; weights.  (us a step, calls in a row, with this, the kept
    // rows and what is looked up ahead, against a sweep and a reduction each for maxima, sums, weights and totals and centres'
    // scores, and every phase loading its own rows: 32 heads with a budget of 128 10.1 / 10.8, 8 heads of 384 17.7 / 20.5,
    // of 512 21.5 / 25.7, 512 heads of 300 17.5 / 19.8; part 2 for 96 heads of 2000 37.8 / 40.3.  float32, then by matrix
    // instructions: 2 heads of 200 19.2 / 26.1, 512 of 300 28.5 / 66.1.)
    constexpr bool kKeep = kAll || G <= 4;                   // (1024 threads have no registers for eight q-heads')
    float x0[kKeep ? kUnroll : 1][G];                        // the first batch's logits
    int ct0[kUnroll];                                        // and its elements' centre tokens
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        if (u * kBlock >= Tn) break;
        ct0[u] = centre_of(pre_rr[u]);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) { m[g] = -INFINITY; inv[g] = 0.f; }
    auto logits_of = [&](int r, float tn, float (&x)[G]) __attribute__((always_inline)) {
        const float rn = r >= 0 ? rn_of[r] : 0.f;
        const float c = a.scale_log2e * (rn > 0.f ? tn / rn : 0.f);
#pragma unroll
        for (int g = 0; g < G; ++g) x[g] = r >= 0 ? c * dot[(size_t)g * Nb + r] : -INFINITY;
    };
    for (int b0 = 0; b0 < Tn; b0 += kBlock * kUnroll) {
        const int j0 = b0 + tid;
        float x[kUnroll][G];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (b0 + u * kBlock >= Tn) break;
            const int j = j0 + u * kBlock;
            int r = pre_rr[u];
            float tn = pre_tn[u], tg = pre_tg[u], tl = pre_tp[u] + pre_tc[u];
            if (b0 != 0) {
                r = j < Tn ? tok_row[j] : -1;
                tn = j < Tn ? tok_norm[j] : 0.f;
                tg = j < Tn ? tok_glo[j] : 0.f;
                tl = j < Tn ? tok_past[j] + tok_cur[j] : 0.f;
            }
            logits_of(r, tn, x[u]);
            if (r >= 0) { tot2[0] += tg; tot2[1] += tl; }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float top = m[g];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                if (b0 + u * kBlock >= Tn) break;
                top = fmaxf(top, x[u][g]);
            }
            const float ref = top > -INFINITY ? top : 0.f;
            float l = inv[g] * exp2_fast(m[g] - ref);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                if (b0 + u * kBlock >= Tn) break;
                l += exp2_fast(x[u][g] - ref);
            }
            m[g] = top; inv[g] = l;
        }
        if (kKeep && b0 == 0) {
#pragma unroll
            for (int u = 0; u < (kKeep ? kUnroll : 1); ++u) {
                if (u * kBlock >= Tn) break;
#pragma unroll
                for (int g = 0; g < G; ++g) x0[u][g] = x[u][g];
            }
        }
    }
    block_softmax<kWaves, G>(m, inv, tot2, vbuf);
    float self_w[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const float M = fmaxf(m[g], self[g]), own = exp2_fast(self[g] - M);
        inv[g] = 1.0f / ((m[g] > -INFINITY ? inv[g] * exp2_fast(m[g] - M) : 0.f) + own);
        m[g] = M;
        self_w[g] = own * inv[g];                            // every thread, same value
        self_tot += self_w[g];
    }
    // Eq. 2 factor on the updated scalars: this step adds one unit of weight per q-head to both totals
    const float s_glo = tot2[0] + (float)G, s_loc = tot2[1] + (float)G;
    const float align = s_glo > 0.f ? s_loc / s_glo : 0.f;
    // accumulate the row into s_Glo and s_Loc^cur (Sec. 3.3); the elements that are class centres' own take part in
    // phase 4: the least important one
    float bv = 0.f;
    int bi = -1;
    for (int b0 = 0; b0 < Tn; b0 += kBlock * kUnroll) {
        const int j0 = b0 + tid;
        int rr[kUnroll], ct[kUnroll];
        float tn[kUnroll], tg[kUnroll], tp[kUnroll], tc[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (b0 + u * kBlock >= Tn) break;
            const int j = j0 + u * kBlock;
            const bool ok = j < Tn;
            if (b0 == 0) { rr[u] = pre_rr[u]; tn[u] = pre_tn[u]; tg[u] = pre_tg[u]; tp[u] = pre_tp[u]; tc[u] = pre_tc[u]; }
            else {
                rr[u] = ok ? tok_row[j] : -1;
                tn[u] = ok ? tok_norm[j] : 0.f;
                tg[u] = ok ? tok_glo[j] : 0.f;
                tp[u] = ok ? tok_past[j] : 0.f;
                tc[u] = ok ? tok_cur[j] : 0.f;
            }
            ct[u] = b0 == 0 ? ct0[u] : centre_of(rr[u]);
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (b0 + u * kBlock >= Tn) break;
            const int j = j0 + u * kBlock;
            if (j >= Tn) break;
            const int r = rr[u];
            float w[G];
            if (r >= 0) {
                float x[G], tot = 0.f;
                if (kKeep && b0 == 0) {
#pragma unroll
                    for (int g = 0; g < G; ++g) x[g] = x0[kKeep ? u : 0][g];
                } else {
                    logits_of(r, tn[u], x);
                }
#pragma unroll
                for (int g = 0; g < G; ++g) { w[g] = exp2_fast(x[g] - m[g]) * inv[g]; tot += w[g]; }
                const float glo = tg[u] + tot, cur = tc[u] + tot;
                tok_glo[j] = glo;
                tok_cur[j] = cur;
                if (j == jo) { old_sc[0] = tn[u]; old_sc[1] = glo; old_sc[2] = tp[u]; old_sc[3] = cur; }
                if (ct[u] == j) {
                    const float sc = fmaxf(glo * align, tp[u] + cur);
                    if (better<true>(sc, r, bv, bi)) { bv = sc; bi = r; }
                }
            } else {
#pragma unroll
                for (int g = 0; g < G; ++g) w[g] = 0.f;
            }
            if (a.attn_opt) {
#pragma unroll
                for (int g = 0; g < G; ++g) a.attn_opt[((size_t)bkv * G + g) * (Tn + 1) + j] = w[g];
            }
        }
    }
    if (a.attn_opt && tid == 0) {
#pragma unroll
        for (int g = 0; g < G; ++g) a.attn_opt[((size_t)bkv * G + g) * (Tn + 1) + Tn] = self_w[g];
    }

    // ---- phase 4: least important class centre (Eq. 2 on the tokens' scalars) ----------
    block_arg<kWaves, true>(bv, bi, fbuf[0], ibuf[0]);             // also: every token's scalars are written

    // ---- phase 3: the oldest window token leaves, the new token takes its ring slot (nothing reads these before the
    // next barrier) ----
    if (row_lane) *reinterpret_cast<frag_t*>(X + ((size_t)ro * kLpr + piece) * 16) = grp == 0 ? new_k : new_v;
    if (tid == 0) {
        tok_pos[jo] = a.seq_len + step; tok_row[jo] = ro; tok_norm[jo] = sh_newnorm;
        tok_glo[jo] = self_tot; tok_past[jo] = 0.f; tok_cur[jo] = self_tot;
        row_norm[ro] = sh_newnorm;
    }
    s_star = max(bi, 0);                                     // block-uniform, in [0, n_imp)
    }   // kDoSoftmax
    if constexpr (kPart == 2) {
        if (row_lane) hand_row[tid] = pre_old;
        if (tid == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) hand[kHandOldSc + i] = old_sc[i];
            hand_i[kHandOldPos] = pre_old_pos;
            hand_i[kHandStar] = s_star;
        }
        return;
    }
    // phase 5's first rows do not depend on the centre that is chosen
    auto load_centres = [&](int base) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            const int s = base + mine + u * kRowsPerPass;
            row_pre[u] = load_frag_or_zero(Kc, ((size_t)s * kLpr + piece) * 16, s < c_end);
        }
    };
    if constexpr (kPart == 5) s_star = hand_i[kHandStar];
    f = kAll && ct_in_lds ? sh_ct[s_star] : entry_tok[s_star];

    // ---- phase 5: its most similar other centre (Eq. 5, cosine of the stored keys) -----
    // Per entry row the dot with the chosen row and the row's own squared norm, as in phase 1.
    if constexpr (kDoCos) {
        frag_t sp;
        if (kAll && s_star < kRowsPerPass * kInFlight) {     // block-uniform: some thread group has the row
#pragma unroll
            for (int u = 0; u < kInFlight; ++u)
                if (mine + u * kRowsPerPass == s_star) star_k[piece] = row_pre[u];
            __syncthreads();
            sp = star_k[piece];
        } else {
            sp = *reinterpret_cast<const frag_t*>(Kc + ((size_t)s_star * kLpr + piece) * 16);
        }
        const float rn_star = row_inv_norm<T>(group_sum<kLpr>(frag_sumsq<T>(sp)));
        for (int base = r_lo; base < c_end; base += kRowsPerPass * kInFlight) {
            if (!kAll || base != r_lo) load_centres(base);
            const frag_t (&fk)[kInFlight] = row_pre;
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                const int s = base + mine + u * kRowsPerPass;
                if (base + u * kRowsPerPass >= c_end) break; // block-uniform
                if (s >= c_end) break;                       // uniform over the row's lanes
                const float d = group_sum<kLpr>(frag_dot<T>(fk[u], sp));
                const float e2 = group_sum<kLpr>(frag_sumsq<T>(fk[u]));
                const float sim = (d * row_inv_norm<T>(e2)) * rn_star;
                if (piece == 0 && s != s_star && better<false>(sim, s, cv, ci)) { cv = sim; ci = s; }
            }
        }
    }   // kDoCos
    block_arg<kWaves, false>(cv, ci, fbuf[1], ibuf[1]);
    if constexpr (kPart == 5) {
        if (tid == 0) { hand[kHandPart + 2 * slice] = cv; hand_i[kHandPart + 2 * slice + 1] = ci; }
        return;
    }
    const bool merged = ci >= 0 && cv > a.tau;
    const int dst = merged ? ci : -1;

    // ---- phase 6: merge at class-centre level, or evict; followers follow --------------
    if (merged && row_lane)
        merge_rows<T>(X + ((size_t)dst * kLpr + piece) * 16, *reinterpret_cast<const frag_t*>(X + ((size_t)s_star * kLpr + piece) * 16), grp == 0,
                      (float)entry_count[s_star], (float)entry_count[dst], row_norm[s_star], row_norm[dst]);
    for (int b0 = 0; b0 < E; b0 += kBlock * kUnroll) {
        int rr[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (b0 + u * kBlock >= E) break;                 // block-uniform
            const int j = b0 + tid + u * kBlock;
            rr[u] = j >= E ? -1 : b0 == 0 ? pre_rr[u] : tok_row[j];
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (b0 + u * kBlock >= E) break;
            const int j = b0 + tid + u * kBlock;
            if (rr[u] != s_star || j == f) continue;
            if (merged) {
                tok_row[j] = dst;
            } else {
                tok_row[j] = -1; tok_pos[j] = -1;
                tok_norm[j] = 0.f; tok_glo[j] = 0.f; tok_past[j] = 0.f; tok_cur[j] = 0.f;
            }
        }
    }
    // the token that left the window is the new centre of entry s_star and takes the
    // departed centre's table element (rows and scalars are written by the lanes, or the wave, that have read them)
    if (row_lane) *reinterpret_cast<frag_t*>(X + ((size_t)s_star * kLpr + piece) * 16) = pre_old;
    if (tid == 0) {
        if (merged) entry_count[dst] += entry_count[s_star];
        entry_count[s_star] = 1;
        row_norm[s_star] = old_sc[0];
        tok_pos[f] = pre_old_pos; tok_row[f] = s_star; tok_norm[f] = old_sc[0];
        tok_glo[f] = old_sc[1]; tok_past[f] = old_sc[2]; tok_cur[f] = old_sc[3];
        if (a.decision_opt) { a.decision_opt[(size_t)bkv * 2] = s_star; a.decision_opt[(size_t)bkv * 2 + 1] = dst; }
        if (a.sim_opt) a.sim_opt[bkv] = ci >= 0 ? cv : -INFINITY;
    }

    // ---- phase 7: a full window of queries: s_Loc^cur becomes s_Loc^past (Sec. 3.3) ----
    if ((step + 1) % W == 0) {                               // block-uniform
        __syncthreads();
        for (int j = tid; j < Tn; j += kBlock) { tok_past[j] = tok_cur[j]; tok_cur[j] = 0.f; }
    }
    // the counter: in the sliced step every block reads the hand-over copy, and a step whose number
    // came with the call reads none
    if (a.step >= 0) {
        if (bkv == 0 && tid == 0) *a.st.step_count = step + 1;
    }
}

__global__ void decode_bump_kernel(int32_t* step_count)
{
    *step_count += 1;
}

// ------------------------------------------------------------------------------------
template <typename T, int D>
static hipError_t launch_decode_init_t(const DecodeInitArgs& a, hipStream_t st)
{
    const int Tn = a.n_imp + a.n_tbm + a.window;
    hipLaunchKernelGGL((decode_init_kernel<T, D>), dim3((Tn + 255) / 256, a.bkv), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_decode_init(const DecodeInitArgs& a, bool f32, hipStream_t st)
{
    if (f32) return a.head_dim == 64 ? launch_decode_init_t<float, 64>(a, st) : launch_decode_init_t<float, 128>(a, st);
    return a.head_dim == 64 ? launch_decode_init_t<bf16_t, 64>(a, st) : launch_decode_init_t<bf16_t, 128>(a, st);
}

// One launch for the choice while what its blocks form more than once -- every block the scores of all centres -- costs less
// than a launch: blocks x centres x (q-heads + 1).  us a step, one launch / two, head size 128:
//    8 heads of 4, budget 2048   1.9 M    16.6 / 18.2        8 heads of 4, 4096   5.2 M   21.4 / 21.0
//   32 heads of 4,        1000   1.8 M    20.2 / 20.7       16 heads of 4, 2048   3.8 M   20.5 / 20.1
//    2 heads of 8,        4000   2.3 M    23.5 / 23.4       32 heads of 8, 1000   3.2 M   25.3 / 24.4
//   32 heads of 1,        2000   3.0 M    19.4 / 19.9       32 heads of 4, 2000   7.4 M   25.3 / 23.2
// (The same with four launches, the scores by the table's slices, the cosines' and the commit's chains not yet shortened:
// 21.1, 23.4, 27.7, 21.4; 24.1, 22.7, 28.0, 25.9.)
constexpr long long kChooseScores = 3000000;
static bool choose_in_one(int heads, int n_imp, int group, int blocks) { return (long long)blocks * heads * n_imp * (group + 1) <= kChooseScores; }
// Threads of the one-launch step: a block of 512 has half the rows and table elements a wave, but pays the rest of the step twice as often.
// (us a step, 256 / 512 threads, head size 128, 4 q-heads, merge ratio 0.5 unless stated: 32 heads of budget 128 9.4 / 10.0, one of 200 at ratio 2
// 12.0 / 11.2, 8 of 256 13.2 / 12.0, of 512 20.1 / 16.6; 128 of 300 15.7 / 13.8.  Before sweeps ended with the table and the new token had a row
// of its own, 256 threads: 10.5, 12.0, 14.2, 21.4; 16.5.)
// In 16 bits at head size 64 with 8 q-heads the dots are most of a wave's work and half as many, and the line lies higher, in rows and in table
// elements: 8 heads, budget / table 300 / 450 14.2 / 14.8, 300 / 900 15.2 / 15.4, 380 / 570 16.0 / 16.0, 420 / 630 16.8 / 16.5, 512 / 768 17.6 / 17.0,
// 256 / 1280 15.2 / 14.8, 400 / 1200 17.6 / 16.3, 512 / 1536 20.6 / 17.8; 32 heads of 200 / 600 13.0 / 14.1, of 380 / 1140 18.3 / 16.9; 256 heads of
// 256 / 512 13.0 / 14.3.  (In float32 200 / 400 15.3 / 15.1, 300 / 900 19.5 / 17.7.)
constexpr int kOneBlockTable = 256, kNarrowRows = 400, kNarrowTable = 1024;
// kWhich: the step kernel's parts (8 = part 0 with 512 threads), 6 = logits, 7 = choice of the centres
template <typename T, int D, int G, int kWhich>
static void launch_decode_group(const DecodeStepArgs& a, hipStream_t st)
{
    if constexpr (kWhich == 6)
        hipLaunchKernelGGL((decode_logits_kernel<D, G>), dim3(a.n_tok_slices, a.bkv), dim3(256), 0, st, a);
    else if constexpr (kWhich == 7) {
        const dim3 toks(a.n_tok_slices, a.bkv), rows(a.n_slices, a.bkv), most(max(a.n_tok_slices, a.n_slices), a.bkv);
        if (choose_in_one(a.bkv, a.n_imp, G, most.x))
            hipLaunchKernelGGL((decode_choose_kernel<D, G, 512, kChoose>), most, dim3(512), 0, st, a);
        else {
            hipLaunchKernelGGL((decode_choose_kernel<D, G, 256, kWeights>), toks, dim3(256), 0, st, a);
            if (hipPeekAtLastError() != hipSuccess) return;
            hipLaunchKernelGGL((decode_choose_kernel<D, G, 256, kCosines>), rows, dim3(256), 0, st, a);
        }
    }
    else {
        constexpr int kPart = kWhich == 8 ? 0 : kWhich;
        constexpr bool kRows = kWhich == 1 || kWhich == 5;      // a block per slice of rows
        constexpr int kBlock = kWhich == 2 ? 1024 : kWhich == 8 ? 512 : 256;
        const size_t lds = kPart == 0 || kPart == 2 ? sizeof(float) * (size_t)(a.lds_floats + a.lds_centres) : 0;
        hipLaunchKernelGGL((decode_step_kernel<T, D, G, kBlock, kPart>), dim3(kRows ? a.n_slices : 1, a.bkv), dim3(kBlock), lds, st, a);
    }
}

template <typename T, int D, int kWhich>
static hipError_t launch_decode_part(const DecodeStepArgs& a, hipStream_t st)
{
    switch (a.group) {
        case 1: launch_decode_group<T, D, 1, kWhich>(a, st); break;
        case 2: launch_decode_group<T, D, 2, kWhich>(a, st); break;
        case 4: launch_decode_group<T, D, 4, kWhich>(a, st); break;
        case 8: launch_decode_group<T, D, 8, kWhich>(a, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Whether the step runs as several launches, and how the rows and (up to kTableHeads heads) the token table are cut.
// f32 rows need twice the operand registers: the validation mode always takes the one-block kernel.
constexpr int kTableHeads = 32;        // figures at the step kernel
bool decode_split(int heads, int budget, int n_imp, int n_tbm, int window, bool f32, DecodeSlices* s)
{
    *s = DecodeSlices{0, 1, 0, 1};
    const int table = n_imp + n_tbm + window;
    if (f32 || (budget <= 512 && table <= 2048)) return false;
    auto cut = [](int n, int* per, int* count) {             // slices of 128, longer ones where that makes too many
        *per = 128;
        while ((n + *per - 1) / *per > kDecodeMaxSlices) *per *= 2;
        *count = (n + *per - 1) / *per;
    };
    if (heads <= kTableHeads) {
        cut(n_imp, &s->rows, &s->n_rows);
        cut(table, &s->toks, &s->n_toks);
    } else {
        cut(budget + 1, &s->rows, &s->n_rows);               // the new key's row included
    }
    return true;
}

int decode_launches(int heads, int group, int budget, int n_imp, int n_tbm, int window, bool f32)
{
    DecodeSlices s;
    if (!decode_split(heads, budget, n_imp, n_tbm, window, f32, &s)) return 1;
    return s.toks > 0 && choose_in_one(heads, n_imp, group, std::max(s.n_toks, s.n_rows)) ? 3 : 4;
}

template <typename T, int D>
static hipError_t launch_decode_step_t(const DecodeStepArgs& a, hipStream_t st)
{
    if (a.slice_rows > 0) {
        if constexpr (sizeof(T) == 2) {
            const bool table = a.tok_slice > 0;
            hipError_t e = table ? launch_decode_part<T, D, 6>(a, st) : launch_decode_part<T, D, 1>(a, st);
            if (e == hipSuccess) e = table ? launch_decode_part<T, D, 7>(a, st) : launch_decode_part<T, D, 2>(a, st);
            if (e == hipSuccess && !table) e = launch_decode_part<T, D, 5>(a, st);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL((decode_commit_kernel<T, D>), dim3(a.bkv), dim3(kCommitBlock), 0, st, a);     // (advances the counter)
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;
        }
    }
    const int table = a.n_imp + a.n_tbm + a.window;
    const bool narrow = sizeof(T) == 2 && D == 64 && a.group == 8 && a.budget <= kNarrowRows && table <= kNarrowTable;
    const bool wide = table > kOneBlockTable && !narrow;
    const hipError_t e = wide ? launch_decode_part<T, D, 8>(a, st) : launch_decode_part<T, D, 0>(a, st);
    // A step whose number came with the call advances the counter itself: only blocks that read the
    // counter need it to stand still until all have (2.7 us of 13.6 a step, 32 heads with a budget of 128).
    if (e != hipSuccess || a.step >= 0) return e;
    hipLaunchKernelGGL(decode_bump_kernel, dim3(1), dim3(1), 0, st, a.st.step_count);
    return hipGetLastError();
}

hipError_t launch_decode_step(const DecodeStepArgs& a, bool f32, hipStream_t st)
{
    if (f32) return a.head_dim == 64 ? launch_decode_step_t<float, 64>(a, st) : launch_decode_step_t<float, 128>(a, st);
    return a.head_dim == 64 ? launch_decode_step_t<bf16_t, 64>(a, st) : launch_decode_step_t<bf16_t, 128>(a, st);
}

}  // namespace ems
