// What the kernels share that run one wave per work item, one wave per SIMD, with a private LDS ring for
// the streamed operand (the score passes, the redundancy statistic): DMA into the ring and its wait
// counts, and the even deal of a launch's stages over the chip's resident waves.
#pragma once

#include <algorithm>
#include <type_traits>

#include "ems_common.h"

namespace ems {

template <int v> using ic = std::integral_constant<int, v>;
constexpr int kXcds = 8;

__device__ __forceinline__ f32x16_t zero_acc()
{
    return f32x16_t{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
}

// ---- staging of the streamed operand: global memory -> LDS without passing through
// registers (global_load_lds_dwordx4), a ring of stages deep.
//
// One instruction moves 64 lanes x 16 bytes into 1 KiB of consecutive LDS; which 16 bytes of
// global memory a lane fetches is free, so rows are stored unpadded with their 16-byte
// chunks XOR-swizzled by the row number: the 16 lanes that read one chunk column of 16
// consecutive rows then hit 16 different bank groups.  Rows past the end of the matrix
// re-read the last row: callers never let such rows contribute (they are masked by
// causality or carry an infinite log-sum-exp).
template <typename T, int D>
__device__ __forceinline__ int swz_key(int row)
{
    return Tile<T, D>::kChunksPerRow >= 16 ? (row & 15) : ((row >> 1) & 7);
}

// One DMA instruction: every lane moves `kBytes` (16 or 4) from base + off (off per lane,
// base wave-uniform) to LDS byte address lds_addr + lane * kBytes (lds_addr wave-uniform;
// the hardware takes it from M0).  Written as inline assembly on purpose: the compiler would
// otherwise make every later LDS read wait for all DMA in flight, which defeats prefetching
// more than one stage ahead.  Completion is tracked by hand with wait_vmem().
template <int kBytes>
__device__ __forceinline__ void dma_to_lds(const void* base, unsigned off, unsigned lds_addr)
{
    const unsigned m0v = __builtin_amdgcn_readfirstlane(lds_addr);
    if (kBytes == 16)
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(m0v) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(base), "s"(m0v) : "memory", "m0");
}

// Four 16-byte DMA instructions under one M0 value: the instruction's immediate offset
// (0, 1024, 2048, 3072) is added to the global address and to the LDS address alike, so
// instruction i moves 1 KiB from base + off_i + 1024 i to LDS lds_addr + 1024 i.  The
// per-lane offsets are passed without the 1024 i term; those of a stage's second (third, ..)
// group of four hold the group's 4 KiB instead, so that all groups share one base.
__device__ __forceinline__ void dma_to_lds_x4(const void* base, unsigned off0, unsigned off1, unsigned off2,
                                              unsigned off3, unsigned lds_addr)
{
    const unsigned m0v = __builtin_amdgcn_readfirstlane(lds_addr);
    asm volatile("s_mov_b32 m0, %5\n\t"
                 "global_load_lds_dwordx4 %0, %4\n\t"
                 "global_load_lds_dwordx4 %1, %4 offset:1024\n\t"
                 "global_load_lds_dwordx4 %2, %4 offset:2048\n\t"
                 "global_load_lds_dwordx4 %3, %4 offset:3072"
                 ::"v"(off0), "v"(off1), "v"(off2), "v"(off3), "s"(base), "s"(m0v) : "memory", "m0");
}

// The same two with the LDS address given as a wave-uniform base plus a compile-time offset: one
// scalar instruction sets M0.
template <int kLdsOff>
__device__ __forceinline__ void dma_to_lds_x4_at(const void* base, unsigned off0, unsigned off1, unsigned off2,
                                                 unsigned off3, unsigned lds_base)
{
    asm volatile("s_add_u32 m0, %5, %6\n\t"
                 "global_load_lds_dwordx4 %0, %4\n\t"
                 "global_load_lds_dwordx4 %1, %4 offset:1024\n\t"
                 "global_load_lds_dwordx4 %2, %4 offset:2048\n\t"
                 "global_load_lds_dwordx4 %3, %4 offset:3072"
                 ::"v"(off0), "v"(off1), "v"(off2), "v"(off3), "s"(base), "s"(lds_base), "n"(kLdsOff) : "memory", "m0", "scc");
}
// One of the four, which go out one by one where an instruction in the middle of others costs less than four in a row.
template <int kLdsOff, int kBoth>
__device__ __forceinline__ void dma_one_to_lds_at(const void* base, unsigned off, unsigned lds_base)
{
    asm volatile("s_add_u32 m0, %2, %3\n\tglobal_load_lds_dwordx4 %0, %1 offset:%4" ::"v"(off), "s"(base), "s"(lds_base), "n"(kLdsOff), "n"(kBoth)
                 : "memory", "m0", "scc");
}
template <int kLdsOff>
__device__ __forceinline__ void dma_dword_to_lds_at(const void* base, unsigned off, unsigned lds_base)
{
    asm volatile("s_add_u32 m0, %2, %3\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(base), "s"(lds_base), "n"(kLdsOff)
                 : "memory", "m0", "scc");
}

// The value itself, made opaque to the optimiser (stops loop-invariant code motion of what is
// computed from it).
__device__ __forceinline__ int opaque_lane(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// The lane's number, formed anew (nothing is kept in registers for it).
__device__ __forceinline__ int lane_here()
{
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

// Tells the compiler that a tuple without a value yet begins its life here (an accumulator set in only
// some branches would otherwise keep its registers through the loops around it).
__device__ __forceinline__ void defined_here(f32x16_t& v) { asm volatile("" : "=v"(v)); }

// A lane's value and that of the lane 32 away, combined (v_permlane32_swap: no LDS round trip, no lane
// address to keep).  The lower half's value is the first operand in both halves.
__device__ __forceinline__ float halves_sum(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float halves_max(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Combined over the four lanes that agree modulo 16 as well.
__device__ __forceinline__ float quarters_sum(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return halves_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}
__device__ __forceinline__ float quarters_max(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return halves_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}

// LDS byte address of a __shared__ object.
__device__ __forceinline__ unsigned lds_address(const void* p)
{
    return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// Wait until at most kOutstanding of this wave's vector-memory operations are in flight
// (they complete in order), leaving the other counters alone.  The counts the kernels pass
// assume that between the DMA of a stage and its wait the wave issues NO other vector-memory
// instruction -- in particular no scratch (spill) load or store: the build rejects a score
// kernel whose compiled form uses scratch memory.
template <int kOutstanding>
__device__ __forceinline__ void wait_vmem()
{
    static_assert(kOutstanding >= 0 && kOutstanding < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kOutstanding) : "memory");
}

// The same wait for "nothing in flight", in the form the compiler can see: used once after
// the stationary operand's ordinary loads, so that the compiler does not re-insert a full
// wait for them in front of their first use inside the main loop.
__device__ __forceinline__ void wait_vmem_all_visible()
{
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0), expcnt and lgkmcnt left alone
}

// One wait for every LDS read in flight, in the form the compiler can see.  Placed well after a
// batch of fragment reads, it replaces the separate wait the compiler would otherwise put in
// front of each fragment's first use (a dozen scalar instructions per stage).
__device__ __forceinline__ void wait_lds_all_visible()
{
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0), vmcnt and expcnt left alone
}

// The cursor of a stream of stages in one source: the address advances by a stage (kStep bytes) until the
// last one is issued (t_left <= 1) and then stays.  Written out: left to the compiler these few scalar
// instructions become several times as many.
template <int kStep>
__device__ __forceinline__ void advance_cursor(int& t_left, const char*& k)
{
    long long ak;
    asm volatile(
        "s_cmp_gt_i32 %[t], 1\n\t"
        "s_cselect_b64 %[ak], %[ks], 0\n\t"
        "s_sub_u32 %[t], %[t], 1"
        : [t] "+s"(t_left), [ak] "=&s"(ak)
        : [ks] "i"(kStep)
        : "scc");
    k += ak;
}


// ---- the even deal.  Launches too short for work queues (a few items per wave, so whole items are
// left over at the end) are cut by stages instead: a head's work is laid out as one line of stages,
// unit (row tile or key tile) after unit, and every wave takes an equal stretch of it, going from one
// unit into the next in its middle.  A stretch leaves its part of a unit's result in slot (wave + unit)
// of the head -- along the line each new part raises one of the two by one, so the slots are distinct --
// and a small kernel adds a unit's parts in order.  A wave's stretch follows from its place in the head
// and the stretch length alone.  Units start at whole trips of the 16-bit interior loops (kTrip),
// so that cuts at multiples of a trip leave no odd stages for the masked loops.  Every unit is preceded
// by `lead` stages that do not exist: what a wave pays for beginning a unit beside its stages (the
// stationary operand's load, 8 us when all waves load at once, and the masked stages, 2.0 us where an
// interior stage takes 1.5: head size 128, measured in the kernels).
constexpr int kStreamRows = 32;            // rows per stage (one MFMA row tile)
constexpr int kTrip = 4;

// First pass: unit u = 32 * kSub query rows, its stages = 32 keys each up to the diagonal's end.
template <int kSub>
struct DealPass1 {
    static constexpr int kAlign = kSub % kTrip == 0 ? kTrip : 1;
    static constexpr int kLead = kSub % kTrip == 0 ? 8 : 2;
    int n_stages, n_units;
    __host__ __device__ explicit DealPass1(int N) : n_stages((N + kStreamRows - 1) / kStreamRows), n_units((n_stages + kSub - 1) / kSub) {}
    __host__ __device__ int start(int u) const { return kSub * (u * (u + 1) / 2) + kLead * u; }
    __host__ __device__ int first(int u) const { return start(u) + kLead; }      // its first real stage
    __host__ __device__ int end(int u) const               // (only the last unit may be short)
    {
        const int n = kSub * (u + 1) < n_stages ? kSub * (u + 1) : n_stages;
        return first(u) + (n + kAlign - 1) / kAlign * kAlign;
    }
    __host__ __device__ int total() const { return end(n_units - 1); }
    __device__ int unit_at(int pos) const                  // the unit that holds stage `pos` of the line
    {
        int lo = 0, hi = n_units;                          // start(lo) <= pos < start(hi)
        while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (start(mid) <= pos) lo = mid; else hi = mid; }
        return lo;
    }
};

// v_mfma_f32_16x16x32_bf16: lane l supplies row (A) / column (B) l % 16, its 16-byte chunk l / 16 of four; register r of the
// accumulator holds row 4 * (l / 16) + r of column l % 16.  It takes the matrix time of the 32x32x16 form and twice its issue
// slots (8 clocks each), but less power, which is what limits the clock where the matrix pipe is busy: alone, on
// random operands, 2050-2130 TFLOP/s at 2.06 GHz against 1750-1830 at 1.75.
__device__ __forceinline__ f32x4_t mma16(const frag_t& a, const frag_t& b, const f32x4_t& c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// A value that is the same in every lane, into a scalar register.
__device__ __forceinline__ int scalar(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Wave of an even deal -> its place: the waves of a head are neighbours on one XCD (and share its L2).
struct DealPlace { int head, wave; };
__device__ __forceinline__ DealPlace deal_place(int heads, int waves)
{
    const int n = heads * waves, per_xcd = (n + kXcds - 1) / kXcds;
    const int i = blockIdx.x / kXcds, w = (int)(blockIdx.x % kXcds) * per_xcd + i;
    if (i >= per_xcd || w >= n) return {-1, 0};
    return {scalar(w / waves), scalar(w % waves)};
}

// Stretch length and waves per head of an even deal of `heads` lines of `total` stages over the
// `resident` waves the chip holds (one per SIMD).  More than one
// round of waves is worth it only where the heads divide the waves badly; a part costs about two and a half stages beside its stages (stationary
// operand, ring start).
inline void deal_over_waves(int resident, long long heads, long long total, int align, int shortest, int* len, int* waves)
{
    double best = 0.;
    for (int rounds = 1; rounds <= 4; ++rounds) {
        const long long per_head = std::max(1ll, (long long)resident * rounds / heads);
        long long l = std::max((long long)shortest, (total + per_head - 1) / per_head);
        l = (l + align - 1) / align * align;
        const long long w = (total + l - 1) / l;
        const double cost = (double)((heads * w + resident - 1) / resident) * ((double)l + 2.5);
        if (rounds == 1 || cost < best) { best = cost; *len = (int)l; *waves = (int)w; }
    }
}

inline long long deal_grid(long long heads, long long waves) { return kXcds * ((heads * waves + kXcds - 1) / kXcds); }


}  // namespace ems
