// Device helpers shared by the triangular-solve kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "hec_dev.h"

namespace hec {

template <typename T> __device__ __forceinline__ T sentinel();
template <> __device__ __forceinline__ double sentinel<double>() { return __longlong_as_double((long long)kSentinel64); }
template <> __device__ __forceinline__ float sentinel<float>() { return __uint_as_float(kSentinel32); }
__device__ __forceinline__ bool is_sentinel(double v) { return __double_as_longlong(v) == (long long)kSentinel64; }
__device__ __forceinline__ bool is_sentinel(float v) { return __float_as_uint(v) == kSentinel32; }

// A right-hand-side value as a kernel publishes it: an input whose bits
// happen to equal the sentinel becomes the canonical quiet NaN, so that no
// input value can stand for "not solved yet" (a row without dependencies
// publishes its right-hand side unchanged).
template <typename T> __device__ __forceinline__ T canon(T v)
{
    return is_sentinel(v) ? __builtin_nan("") : v;
}
template <> __device__ __forceinline__ float canon<float>(float v)
{
    return is_sentinel(v) ? __builtin_nanf("") : v;
}

// Right-hand side times the reciprocal diagonal, rounded on its own (never
// contracted into the first multiply-add), identically in every kernel.
__device__ __forceinline__ double scale_rhs(double b, double d)
{
#pragma clang fp contract(off)
    return b * d;
}
__device__ __forceinline__ float scale_rhs(float b, float d)
{
#pragma clang fp contract(off)
    return b * d;
}

}  // namespace hec
