// Packed matrix rows and LDS addressing, shared by the kernels that keep the
// solution in LDS.
#pragma once

#include "tri_dev.h"

namespace hec {

using BufRsrc = __amdgpu_buffer_rsrc_t;

// A value of LDS by its byte offset.  Kernels that use this have no static
// LDS, so their dynamic LDS, which starts with the value area, starts at LDS
// address 0 (checked at launch): an offset is an address, with no base to add
// on the dependency chain.
template <typename T> using LdsPtr = __attribute__((address_space(3))) T *;
template <typename T> __device__ __forceinline__ T lds_at(unsigned off)
{
    return __hip_atomic_load((LdsPtr<T>)(uintptr_t)off, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T> __device__ __forceinline__ void lds_set(unsigned off, T v)
{
    __hip_atomic_store((LdsPtr<T>)(uintptr_t)off, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// A row as it is stored: W values, then W 16-bit LDS value rows, in 16-byte
// chunks and a remainder of 0..2 dwords, each chunk an array over the rows.
// Three dwords are padded to a chunk.  (RowRecord on the host.)
template <typename T, int W> struct RowRec {
    static constexpr int V = W * (int)sizeof(T) / 4;  // dwords of values
    static constexpr int NB = V + (W + 1) / 2;
    static constexpr int CH = NB / 4 + (NB % 4 == 3 ? 1 : 0);
    static constexpr int RE = NB % 4 == 3 ? 0 : NB % 4;
    static constexpr int ND = 4 * CH + RE;
    static constexpr int LOADS = CH + (RE > 0 ? 1 : 0);
};

template <typename T, int W> using RowRegs = uint32_t[RowRec<T, W>::ND];

// The record at byte offset vo of its first chunk from `base`; chunk c lies
// c * ld * 16 bytes behind, the remainder (a quarter or half as wide) at rbase.
template <typename T, int W>
__device__ __forceinline__ void row_load(RowRegs<T, W> &d, BufRsrc rsrc, unsigned ld,
                                         unsigned base, unsigned rbase, unsigned vo)
{
    using Rec = RowRec<T, W>;
#pragma unroll
    for (int c = 0; c < Rec::CH; ++c) {
        auto v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)vo, (int)(base + c * ld * 16u), 0);
        d[4 * c] = v[0];
        d[4 * c + 1] = v[1];
        d[4 * c + 2] = v[2];
        d[4 * c + 3] = v[3];
    }
    if constexpr (Rec::RE == 1) d[4 * Rec::CH] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)(vo / 4u), (int)rbase, 0);
    if constexpr (Rec::RE == 2) {
        auto v = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)(vo / 2u), (int)rbase, 0);
        d[4 * Rec::CH] = v[0];
        d[4 * Rec::CH + 1] = v[1];
    }
}

template <typename T, int W> __device__ __forceinline__ T row_val(const RowRegs<T, W> &d, int e)
{
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, (unsigned long long)d[2 * e] | ((unsigned long long)d[2 * e + 1] << 32));
    else
        return __builtin_bit_cast(T, d[e]);
}

// LDS byte offset of ELL slot e: its value row times ROWB bytes.  One
// multiply-add on a half of the packed dword.
template <typename T, int W, unsigned ROWB>
__device__ __forceinline__ unsigned row_off(const RowRegs<T, W> &d, int e)
{
    const unsigned p = d[RowRec<T, W>::V + e / 2];
    unsigned r;
    if (e & 1) asm volatile("v_mad_u32_u16 %0, %1, %2, 0 op_sel:[1,0,0,0]" : "=v"(r) : "v"(p), "n"(ROWB));
    else asm volatile("v_mad_u32_u16 %0, %1, %2, 0" : "=v"(r) : "v"(p), "n"(ROWB));
    return r;
}
// The same for a row size that is a launch argument, plus an offset in the row.
template <typename T, int W>
__device__ __forceinline__ unsigned row_off(const RowRegs<T, W> &d, int e, unsigned rowb, unsigned add)
{
    const unsigned p = d[RowRec<T, W>::V + e / 2];
    unsigned r;
    if (e & 1) asm volatile("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(r) : "v"(p), "s"(rowb), "v"(add));
    else asm volatile("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(r) : "v"(p), "s"(rowb), "v"(add));
    return r;
}

}  // namespace hec
