// Row-wise helpers shared by the merge, expansion and decode kernels: a cache row of D
// elements is handled as 16-byte pieces, one per lane.
#pragma once

#include "ems_common.h"

namespace ems {

// Dot product of the 8 bf16 elements of two 16-byte row pieces, f32 accumulation.  v_dot2 keeps subnormal sums (the
// norms of rows of 2^-75 come out as by single multiply-adds), and the norms are as close to 64 bits: 3.3e-8 either way.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float dot8_bf16(const frag_t& x, const frag_t& y)
{
    const bf16x8_t a = __builtin_bit_cast(bf16x8_t, x), b = __builtin_bit_cast(bf16x8_t, y);
    float acc = 0.f;
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 0, 1), __builtin_shufflevector(b, b, 0, 1), acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 2, 3), __builtin_shufflevector(b, b, 2, 3), acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 4, 5), __builtin_shufflevector(b, b, 4, 5), acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 6, 7), __builtin_shufflevector(b, b, 6, 7), acc, false);
    return acc;
}

// dot product of two 16-byte fragments, in f32
template <typename T> __device__ __forceinline__ float frag_dot(const frag_t& x, const frag_t& y);
template <> __device__ __forceinline__ float frag_dot<bf16_t>(const frag_t& x, const frag_t& y) { return dot8_bf16(x, y); }
template <> __device__ __forceinline__ float frag_dot<float>(const frag_t& x, const frag_t& y)
{
    const f32x4_t a = __builtin_bit_cast(f32x4_t, x), b = __builtin_bit_cast(f32x4_t, y);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) s = __builtin_fmaf(a[i], b[i], s);
    return s;
}

// sum of squares of the 16-byte fragment's elements, in f32
template <typename T> __device__ __forceinline__ float frag_sumsq(const frag_t& f);
template <> __device__ __forceinline__ float frag_sumsq<bf16_t>(const frag_t& f) { return dot8_bf16(f, f); }
template <> __device__ __forceinline__ float frag_sumsq<float>(const frag_t& f)
{
    const f32x4_t v = __builtin_bit_cast(f32x4_t, f);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) s = __builtin_fmaf(v[i], v[i], s);
    return s;
}

__device__ __forceinline__ float inv_norm(float sumsq) { return sumsq > 0.f ? 1.0f / sqrtf(sumsq) : 0.f; }

// The same for a row of T by the hardware's reciprocal square root (1 ulp), which is not made for the smallest
// values.  Similarities against 64 bits, 4200 rows of 128: 6.2e-8 rms with it, 6.4e-8 with two rounded steps.
// Float32 rows, the mode that checks the other, add a Newton step with the product's rounding carried along
// (half an ulp and a little; the two rounded steps made the search 5-10 % slower).
template <typename T>
__device__ __forceinline__ float row_inv_norm(float sumsq)
{
    if (!(sumsq >= 0x1p-100f && sumsq <= 0x1p100f)) return inv_norm(sumsq);
    const float y = __builtin_amdgcn_rsqf(sumsq);
    if constexpr (sizeof(T) == 2) return y;
    const float h = sumsq * y, low = __builtin_fmaf(sumsq, y, -h);
    const float e = __builtin_fmaf(-low, y, __builtin_fmaf(-h, y, 1.f));      // 1 - sumsq y^2
    return __builtin_fmaf(0.5f * y, e, y);
}

template <typename T> struct Pack;
template <> struct Pack<bf16_t> {
    static constexpr int kElems = 8;
    static __device__ __forceinline__ void unpack(const frag_t& f, float (&x)[8])
    {
        const bf16x8_t v = __builtin_bit_cast(bf16x8_t, f);
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = (float)v[i];
    }
    static __device__ __forceinline__ frag_t pack(const float (&x)[8])
    {
        bf16x8_t v;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (bf16_t)x[i];      // round to nearest even
        return __builtin_bit_cast(frag_t, v);
    }
};
template <> struct Pack<float> {
    static constexpr int kElems = 4;
    static __device__ __forceinline__ void unpack(const frag_t& f, float (&x)[4])
    {
        const f32x4_t v = __builtin_bit_cast(f32x4_t, f);
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = v[i];
    }
    static __device__ __forceinline__ frag_t pack(const float (&x)[4])
    {
        f32x4_t v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = x[i];
        return __builtin_bit_cast(frag_t, v);
    }
};

// ---- DPP lane permutations (ALU latency, no LDS round trip)
template <int kCtrl>
__device__ __forceinline__ float dpp_f(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kCtrl, 0xf, 0xf, false));
}
template <int kCtrl>
__device__ __forceinline__ int dpp_i(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, kCtrl, 0xf, 0xf, false);
}
constexpr int kDppXor1 = 0xB1;         // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;         // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;  // lane i <-> 7 - i inside each group of 8
constexpr int kDppMirror = 0x140;      // lane i <-> 15 - i inside each row of 16

template <bool kMax> __device__ __forceinline__ float comb(float a, float b) { return kMax ? fmaxf(a, b) : a + b; }
__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}


// Sum over the kLpr consecutive lanes that hold one row (kLpr = 8, 16 or 32); every lane of
// the group gets the total.
template <int kLpr>
__device__ __forceinline__ float group_sum(float v)
{
    v += dpp_f<kDppXor1>(v);
    v += dpp_f<kDppXor2>(v);
    v += dpp_f<kDppHalfMirror>(v);
    if constexpr (kLpr >= 16) v += dpp_f<kDppMirror>(v);
    if constexpr (kLpr >= 32) v += __shfl_xor(v, 16);
    return v;
}

}  // namespace ems
