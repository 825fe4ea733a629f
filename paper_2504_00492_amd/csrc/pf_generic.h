// What the bodies of the generic kernel share (pf_generic.hip, pf_generic_block.h).
#pragma once
#include "pf_common.h"

namespace pf {

template <typename T> __device__ __forceinline__ float as_f32(T v);
template <> __device__ __forceinline__ float as_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float as_f32<uint16_t>(uint16_t v) { return bf16_bits_to_f32(v); }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ uint16_t from_f32<uint16_t>(float v)
{
    const bf16 b = (bf16)v;
    return __builtin_bit_cast(uint16_t, b);
}

template <typename T> struct GenericArgs {
    const T *Q, *K, *V, *beta;
    const float *S0;
    T *O;
    float *SL;
    int heads, L, dk, dv, r, t0, product;
};

}  // namespace pf
