// Row accesses of the vector blocks.
#pragma once

#include "device.hpp"

namespace ftlm {

// Loads/stores VB consecutive elements with the widest naturally aligned
// vector access (the host only picks a vector width whose alignment holds),
// as global-memory accesses.
template <typename T, int N>
using VecT = T __attribute__((ext_vector_type(N)));

template <typename T, int VB>
__device__ __forceinline__ void load_row(const T* __restrict__ p, T (&v)[VB]) {
    if constexpr (sizeof(T) == 4 && VB % 4 == 0) {
#pragma unroll
        for (int i = 0; i < VB; i += 4) {
            const VecT<T, 4> q = *(const FTLM_GLOBAL VecT<T, 4>*)(p + i);
            v[i] = q.x; v[i + 1] = q.y; v[i + 2] = q.z; v[i + 3] = q.w;
        }
    } else if constexpr (VB % 2 == 0) {
#pragma unroll
        for (int i = 0; i < VB; i += 2) {
            const VecT<T, 2> q = *(const FTLM_GLOBAL VecT<T, 2>*)(p + i);
            v[i] = q.x; v[i + 1] = q.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < VB; ++i) v[i] = *gptr(p + i);
    }
}

template <typename T, int VB>
__device__ __forceinline__ void store_row(T* __restrict__ p, const T (&v)[VB]) {
    if constexpr (sizeof(T) == 4 && VB % 4 == 0) {
#pragma unroll
        for (int i = 0; i < VB; i += 4) {
            const VecT<T, 4> q = {v[i], v[i + 1], v[i + 2], v[i + 3]};
            *(FTLM_GLOBAL VecT<T, 4>*)(p + i) = q;
        }
    } else if constexpr (VB % 2 == 0) {
#pragma unroll
        for (int i = 0; i < VB; i += 2) {
            const VecT<T, 2> q = {v[i], v[i + 1]};
            *(FTLM_GLOBAL VecT<T, 2>*)(p + i) = q;
        }
    } else {
#pragma unroll
        for (int i = 0; i < VB; ++i) *gptr(p + i) = v[i];
    }
}

// Fourth word of a raw buffer resource on gfx9: data format 32 bits (a zero
// format makes every load return 0), no stride, no swizzle.
constexpr int kBufferWord3 = 0x00020000;

template <typename T>
__device__ __forceinline__ T bond_coef(const BondTable& B, int b) {
    if constexpr (sizeof(T) == 4) return B.coef_f[b];
    else return B.coef_d[b];
}

}  // namespace ftlm
