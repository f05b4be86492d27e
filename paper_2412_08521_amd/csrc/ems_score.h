// What the two score passes share, whatever their element type (score.hip: 16 bits, score_f32.hip: float32): how a
// wave comes to its work items, and the plain form of a tile.
#pragma once

#include "ems_common.h"
#include "ems_kernels.h"
#include "ems_stream.h"

namespace ems {

// The hardware deals workgroups to the 8 XCDs (each with its own L2) round-robin in launch
// order: block b runs on XCD b % 8.  First pass: work is cut into groups of `per_group`
// consecutive work items that stream the same operand; group g belongs to XCD g % 8 so that the
// group shares one L2.  Returns the linear index of the k-th work item of XCD `xcd`, or -1 for
// padding.
__device__ __forceinline__ int xcd_work_item(int n_groups, int per_group, int xcd, int k)
{
    const int group = (k / per_group) * kXcds + xcd;
    return group < n_groups ? group * per_group + k % per_group : -1;
}

// ---- work queues.  The XCDs of one chip do not run at the same speed (a few percent apart under
// this load), and the hardware deals workgroups to them in fixed turns, so a launch whose work is
// bound to block indices ends when the slowest XCD ends, with the re-dispatch of a workgroup per
// item on top.  In long launches a wave therefore stays resident and takes its work items at run
// time, one integer atomic per item; which wave computes an item has no influence on the item's
// result.
// Second pass: from the queue of its XCD (items that stream the same operand stay on one L2)
// and, once that is empty, from a pool of the lightest items that every XCD draws from.  Returns
// the item's index in its queue (pool = true: in the pool), or -1 when both are empty.
__device__ __forceinline__ int take_work_item(int* cursors, int n_local, int n_pool, bool& pool)
{
    int k = -1, from_pool = 0;
    if (threadIdx.x == 0) {
        if (n_local > 0) {
            k = atomicAdd(&cursors[blockIdx.x % kXcds], 1);
            if (k >= n_local) k = -1;
        }
        if (k < 0 && n_pool > 0) {
            k = atomicAdd(&cursors[kXcds], 1);
            from_pool = 1;
            if (k >= n_pool) k = -1;
        }
    }
    pool = __builtin_amdgcn_readfirstlane(from_pool) != 0;
    return __builtin_amdgcn_readfirstlane(k);
}

// First pass: every XCD has a queue (its items in the fixed order of xcd_work_item, padding
// included); a wave whose own queue is empty goes on with the next item of another XCD's queue,
// so the faster XCDs help the slower ones finish.  Returns the item's index in the queue of XCD
// `from`, or -1 when every queue is empty.
__device__ __forceinline__ int take_or_steal(int* cursors, int n_per_queue, int& from)
{
    int k = -1, q = 0;
    if (threadIdx.x == 0) {
        const int own = blockIdx.x % kXcds;
        for (int d = 0; d < kXcds && k < 0; ++d) {
            q = (own + d) % kXcds;
            k = atomicAdd(&cursors[q], 1);
            if (k >= n_per_queue) k = -1;
        }
    }
    from = __builtin_amdgcn_readfirstlane(q);
    return __builtin_amdgcn_readfirstlane(k);
}

// Pass 2: key tiles at or below the diagonal of row chunks 0..I, per (batch, kv-head): chunk I'
// has min(n_key_tiles, (I' + 1) * r) of them, r = chunk rows / keys per tile.
__host__ __device__ inline long long p2_items_upto(int I, int r, int n_key_tiles)
{
    const long long n = I + 1;
    const long long whole = n < n_key_tiles / r ? n : n_key_tiles / r;    // chunks whose count is not capped
    return r * whole * (whole + 1) / 2 + (n - whole) * n_key_tiles;
}

// Second pass: unit u = 32 * kSub keys, its stages = 32 query rows each (of every q-head of the group)
// from the diagonal on.
template <int kSub>
struct DealPass2 {
    int n_units, rows_all, lead;                           // rows_all: stages of unit 0, padding included
    __host__ __device__ DealPass2(int N, int group)
    {
        const int n_stages = (N + kStreamRows - 1) / kStreamRows;
        n_units = (n_stages + kSub - 1) / kSub;
        const int a = align(group);
        rows_all = (n_stages + a - 1) / a * a;
        // (the operand's load is paid once for the q-heads of the group, the masked stages by each)
        lead = kSub % kTrip ? (group == 1 ? 2 : 1) : ((2 * group + 5 + group / 2) / group + a - 1) / a * a;
    }
    // a stretch that starts and ends at these multiples holds whole trips (of stages x q-heads)
    static __host__ __device__ int align(int group) { return kSub % kTrip ? 1 : group % 4 == 0 ? 1 : group % 2 == 0 ? 2 : kTrip; }
    __host__ __device__ int start(int u) const { return u * (rows_all + lead) - kSub * (u * (u - 1) / 2); }
    __host__ __device__ int first(int u) const { return start(u) + lead; }
    __host__ __device__ int end(int u) const { return start(u + 1); }
    __host__ __device__ int total() const { return start(n_units); }
    __device__ int unit_at(int pos) const
    {
        int lo = 0, hi = n_units;
        while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (start(mid) <= pos) lo = mid; else hi = mid; }
        return lo;
    }
};

// The work items of a wave of the second pass: (row chunk I, (batch, kv-head), key tile J at or below the chunk's diagonal),
// heaviest chunks first.  An XCD's queue holds the chunks from the top down to p2_split for its share of the heads (head =
// XCD + 8 m), key tiles innermost, so that the waves of an XCD stream the same query rows; the chunks below p2_split, all
// heads, are the pool.  Long launches: a wave stays and takes item after item until the queues are empty -- the exit every wave
// reaches (the cursors only grow); between two items nothing of the wave is in flight.  Shorter ones: the wave's stretch of an
// even deal, one part of a key tile after the other.  When the heads do not divide over the XCDs there are no
// queues: the groups (I, head) are dealt to the XCDs in turn and every block has one item, fixed by its index.
template <int kSub, bool kDeal>
struct Pass2Items {
    static constexpr int kKeys = 32 * kSub;
    const ScoreArgs& a;
    const DealPass2<kSub> deal;
    DealPlace place{-1, 0};
    int pos = 0, pos_end = 0;
    bool first = true;
    int I = 0, J = 0, bkv = 0, r_begin = 0, r_end = 0;         // the item: rows [r_begin, r_end), r_begin a multiple of 32

    __device__ __forceinline__ explicit Pass2Items(const ScoreArgs& args) : a(args), deal(args.seq_len, args.q_heads / args.kv_heads)
    {
        if constexpr (kDeal) {
            place = deal_place(a.batch * a.kv_heads, a.p2_waves);
            if (place.head < 0) return;
            pos = place.wave * a.p2_len;
            pos_end = scalar(min(pos + a.p2_len, deal.total()));
        }
    }
    // the wave's next item with rows; false: it has none left
    __device__ __forceinline__ bool next()
    {
        const int N = a.seq_len;
        for (; first || kDeal || a.q_dynamic;) {
            first = false;
            if constexpr (kDeal) {
                if (pos >= pos_end) return false;
                J = scalar(deal.unit_at(pos));
                bkv = place.head;
                const int u0 = deal.first(J), to = min(pos_end, deal.end(J));
                r_begin = scalar(J * kKeys + (max(pos, u0) - u0) * kStreamRows);
                r_end = scalar(min(J * kKeys + (to - u0) * kStreamRows, N));
                pos = scalar(to);
            } else {
                const int n_key_tiles = (N + kKeys - 1) / kKeys, n_chunks = a.n_chunks, R = a.chunk_rows, BKV = a.batch * a.kv_heads;
                if (a.q_share == 0) {
                    int bid = xcd_work_item(BKV * n_chunks, n_key_tiles, blockIdx.x % kXcds, blockIdx.x / kXcds);
                    if (bid < 0) return false;
                    J = bid % n_key_tiles; bid /= n_key_tiles;
                    bkv = bid % BKV;
                    I = n_chunks - 1 - bid / BKV;
                } else {
                    bool pool;
                    const int k = take_work_item(a.queue, a.p2_local, a.p2_pool, pool);
                    if (k < 0) return false;
                    const int r_tiles = R / kKeys;
                    const int top = pool ? a.p2_split - 1 : n_chunks - 1;
                    const long long per = pool ? BKV : a.q_share;       // heads per chunk in this queue
                    const long long upto_top = p2_items_upto(top, r_tiles, n_key_tiles);
                    int lo = pool ? 0 : a.p2_split, hi = top;           // the chunk whose items include k: the smallest I with before(I) <= k
                    while (lo < hi) {
                        const int mid = (lo + hi) >> 1;
                        if (per * (upto_top - p2_items_upto(mid, r_tiles, n_key_tiles)) <= k) hi = mid; else lo = mid + 1;
                    }
                    I = lo;
                    const int rem = (int)(k - per * (upto_top - p2_items_upto(I, r_tiles, n_key_tiles)));
                    const int cnt = min(n_key_tiles, (I + 1) * r_tiles);
                    J = rem % cnt;
                    bkv = pool ? rem / cnt : (int)(blockIdx.x % kXcds) + kXcds * (rem / cnt);
                }
                r_begin = max(I * R, J * kKeys);                        // both multiples of 32
                r_end = min((I + 1) * R, N);
            }
            if (r_begin < r_end) return true;               // (else: pair above the diagonal, of which the queues hold none, or padding)
        }
        return false;
    }
    // where the item's sums go: key kj to out_glo[kj] and, where out_loc is set, out_loc[kj]
    __device__ __forceinline__ void outputs(float*& out_glo, float*& out_loc) const
    {
        const int N = a.seq_len;
        out_loc = nullptr;
        if constexpr (kDeal) {
            const ptrdiff_t at = ((ptrdiff_t)bkv * (a.p2_waves + deal.n_units) + place.wave + J) * kKeys - J * kKeys;
            out_glo = a.part_glo + at;
            if (r_end > N - a.window) out_loc = a.part_loc + at;
        } else {
            const int n_chunks = a.n_chunks, loc_chunk0 = a.loc_chunk0;
            out_glo = n_chunks == 1 ? a.s_glo + (size_t)bkv * N : a.part_glo + ((size_t)bkv * n_chunks + I) * N;
            if (n_chunks == 1) out_loc = a.s_loc + (size_t)bkv * N;
            else if (I >= loc_chunk0) out_loc = a.part_loc + ((size_t)bkv * (n_chunks - loc_chunk0) + (I - loc_chunk0)) * N;
        }
    }
};

// The same for the first pass: row tile rt of q-head g of the group bkv (= b * kv_heads + kv), key stages [t0, t1).
// (p1_by_block: one item per block, by its index.)
template <int kSub, bool kDeal>
struct Pass1Items {
    static constexpr int kRows = 32 * kSub;
    const ScoreArgs& a;
    const DealPass1<kSub> deal;
    DealPlace place{-1, 0};
    int pos = 0, pos_end = 0, q_head = 0;
    bool first = true;
    int rt = 0, bkv = 0, g = 0, t0 = 0, t1 = 0;

    __device__ __forceinline__ explicit Pass1Items(const ScoreArgs& args) : a(args), deal(args.seq_len)
    {
        if constexpr (kDeal) {
            // neighbours are the q-heads of a group on the same stretch: they stream the same keys, through one L2
            const int G = a.q_heads / a.kv_heads;
            place = deal_place(a.batch * a.kv_heads, a.p1_waves * G);
            if (place.head < 0) return;
            q_head = scalar(place.wave % G); place.wave = scalar(place.wave / G);
            pos = place.wave * a.p1_len;
            pos_end = scalar(min(pos + a.p1_len, deal.total()));
        }
    }
    __device__ __forceinline__ bool next()
    {
        const int N = a.seq_len, G = a.q_heads / a.kv_heads, n_row_tiles = (N + kRows - 1) / kRows;
        for (;;) {
            if constexpr (kDeal) {
                if (pos >= pos_end) return false;
                rt = scalar(deal.unit_at(pos));
                g = q_head; bkv = place.head;
                const int u0 = deal.first(rt), to = min(pos_end, deal.end(rt));
                t0 = scalar(max(pos, u0) - u0); t1 = scalar(to - u0);
                pos = scalar(to);
                if (t0 >= t1) continue;                     // before the unit's first stage
            } else {
                // the first item goes by the wave's place: a thousand waves would wait for one cache line of cursors
                int from_xcd = blockIdx.x % kXcds, k_item = blockIdx.x / kXcds;
                if (!first && a.p1_by_block) return false;
                if (!first || k_item >= a.p1_local) k_item = take_or_steal(a.queue + (kXcds + 1), a.p1_local, from_xcd);
                first = false;
                if (k_item < 0) return false;
                int bid = xcd_work_item(a.p1_groups, a.p1_per_group, from_xcd, k_item);
                if (bid < 0) continue;                      // padding
                g = bid % G; bid /= G;
                const int BKV = a.batch * a.kv_heads;
                if (a.p1_groups == BKV) { rt = n_row_tiles - 1 - (bid % n_row_tiles); bkv = bid / n_row_tiles; }
                else { bkv = bid % BKV; rt = n_row_tiles - 1 - (bid / BKV); }   // heaviest row tiles first
                t1 = kSub * (rt + 1);
            }
            t1 = min(t1, (min(N, (rt + 1) * kRows) + kStreamRows - 1) / kStreamRows);   // the stages the row tile can see
            return true;
        }
    }
};

// A stretch of an even deal can be as long as a whole row or column.  After kFoldKeys keys (first pass), or kFoldRows
// rows of every q-head of the group (second), a running sum is added to the sum of those before it, so that
// small weights are not lost against a large sum.  (1 x 4 heads over 1, 8192: column sums off by 3.8e-7 without, 0.7e-7.)
constexpr int kFoldKeys = 2048, kFoldRows = 512;
// sum of the 16 accumulator-derived values with four independent partial sums
__device__ __forceinline__ float sum16(const float (&p)[16])
{
    float s0 = p[0], s1 = p[1], s2 = p[2], s3 = p[3];
#pragma unroll
    for (int r = 4; r < 16; r += 4) { s0 += p[r]; s1 += p[r + 1]; s2 += p[r + 2]; s3 += p[r + 3]; }
    return (s0 + s1) + (s2 + s3);
}

__device__ __forceinline__ float max16(const f32x16_t& acc)
{
    float t0 = fmaxf(fmaxf(acc[0], acc[1]), acc[2]);
    float t1 = fmaxf(fmaxf(acc[3], acc[4]), acc[5]);
    float t2 = fmaxf(fmaxf(acc[6], acc[7]), acc[8]);
    float t3 = fmaxf(fmaxf(acc[9], acc[10]), acc[11]);
    float t4 = fmaxf(fmaxf(acc[12], acc[13]), acc[14]);
    t0 = fmaxf(fmaxf(t0, t1), t2);
    t3 = fmaxf(fmaxf(t3, t4), acc[15]);
    return fmaxf(t0, t3);
}

// A sum above `limit` gives its exponent to its reference; what the sum of reference and exponent loses in
// rounding stays with it.
__device__ __forceinline__ void give_exponent(float& m, float& l, float limit)
{
    const int up = l > limit ? __builtin_amdgcn_frexp_expf(l) : 0;
    const float to = m + (float)up, part = to - m;
    const float lost = up ? (m - (to - part)) + ((float)up - part) : 0.f;      // (m may be infinite where up is 0)
    l = __builtin_amdgcn_ldexpf(l, -up) * exp2_fast(lost);
    m = to;
}

// One 32-key x 32-query tile of the online softmax; it may cross the diagonal.
template <typename T, int D>
__device__ __forceinline__ void pass1_tile(const frag_t (&ak)[Tile<T, D>::kFrags],
                                           const frag_t (&bq)[Tile<T, D>::kFrags],
                                           float& m_run, float& l_run, float c,
                                           int key0, int qi, int half)
{
    f32x16_t acc = zero_acc();
#pragma unroll
    for (int f = 0; f < Tile<T, D>::kFrags; ++f) mma<T>(acc, ak[f], bq[f]);
#pragma unroll
    for (int r = 0; r < 16; ++r)
        if (key0 + acc_row(r, half) > qi) acc[r] = -INFINITY;
    const float tmax = max16(acc);
    const float m_new = fmaxf(m_run, tmax * c);
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    float p[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) p[r] = exp2_fast(__builtin_fmaf(acc[r], c, -m_use));
    l_run = __builtin_fmaf(l_run, exp2_fast(m_run - m_use), sum16(p));
    m_run = m_new;
}

// One 32-row x 32-key tile of the edge loop: weights added into the lane's column sums; the
// tile may cross the diagonal and may hold last-window rows.
template <typename T, int D>
__device__ __forceinline__ void stream_edge_tile(const frag_t (&aq)[Tile<T, D>::kFrags],
                                                 const frag_t (&bk)[Tile<T, D>::kFrags],
                                                 const f32x16_t& lse_v, float c, float& glo, float& loc,
                                                 int row0, int kj, int half, int win0)
{
    constexpr int kFrags = Tile<T, D>::kFrags;
    f32x16_t acc = zero_acc();
    float p[16];
#pragma unroll
    for (int f = 0; f < kFrags; ++f) mma<T>(acc, aq[f], bk[f]);
#pragma unroll
    for (int r = 0; r < 16; ++r) p[r] = exp2_fast(__builtin_fmaf(acc[r], c, -lse_v[r]));
#pragma unroll
    for (int r = 0; r < 16; ++r)
        if (row0 + acc_row(r, half) < kj) p[r] = 0.f;
    glo += sum16(p);
    if (row0 + 31 >= win0) {                               // wave-uniform
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (row0 + acc_row(r, half) < win0) p[r] = 0.f;
        loc += sum16(p);
    }
}

// The interior loops' DMA cursor, one step: source address `q` advances by a stage (kQStep bytes), at
// the last stage of a head (h_left == 1 of per_head) by q_jump instead, and not at all once the
// last stage of all is issued (t_left <= 1); `l` likewise with kLStep / l_jump.  Written out: left
// to the compiler these few selects become several times as many instructions, part of them on
// the vector ALU.
template <int kQStep, int kLStep>
__device__ __forceinline__ void advance_cursor(int& h_left, int& t_left, const char*& q, const char*& l, int per_head,
                                               long long q_jump, long long l_jump)
{
    long long aq, al;
    asm volatile(
        "s_cmp_eq_u32 %[h], 1\n\t"
        "s_cselect_b64 %[aq], %[qj], %[qs]\n\t"
        "s_cselect_b64 %[al], %[lj], %[ls]\n\t"
        "s_cselect_b32 %[h], %[ph], %[h]\n\t"
        "s_sub_u32 %[h], %[h], 1\n\t"
        "s_cmp_gt_i32 %[t], 1\n\t"
        "s_cselect_b64 %[aq], %[aq], 0\n\t"
        "s_cselect_b64 %[al], %[al], 0\n\t"
        "s_sub_u32 %[t], %[t], 1"
        : [h] "+s"(h_left), [t] "+s"(t_left), [aq] "=&s"(aq), [al] "=&s"(al)
        : [qj] "s"(q_jump), [lj] "s"(l_jump), [ph] "s"(per_head + 1), [qs] "i"(kQStep), [ls] "i"(kLStep)
        : "scc");
    q += aq;
    l += al;
}

// What score.hip's launchers start in place of its own kernels: the passes by 16x16x32 products (score_m16.hip), the float32
// passes (score_f32.hip).
constexpr int kSubBf16 = 8;            // 32-wide subtiles of the stationary operand per wave
void start_pass1_m16(const ScoreArgs& a, bool deal, unsigned grid, hipStream_t st);
void start_pass2_m16(const ScoreArgs& a, unsigned grid, hipStream_t st);      // (an even deal)
constexpr int kSubF32 = 2;             // 32-wide subtiles of the stationary operand per wave
void start_pass1_f32(const ScoreArgs& a, bool deal, unsigned grid, hipStream_t st);
void start_pass2_f32(const ScoreArgs& a, bool deal, unsigned grid, hipStream_t st);

}  // namespace ems
