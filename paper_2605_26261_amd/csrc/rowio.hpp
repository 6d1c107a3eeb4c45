// Row accesses of the vector blocks.
#pragma once

#include "kernels.hpp"

namespace ftlm {

// Loads/stores VB consecutive elements with 16- or 8-byte accesses to global
// memory, which need the alignment of one element only (rows of 5 or 7 columns
// begin anywhere).
template <typename T, int N>
struct VecOf {
    typedef T type __attribute__((ext_vector_type(N), aligned(sizeof(T))));
};
template <typename T, int N>
using VecT = typename VecOf<T, N>::type;

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

// No infinity and no NaN among VB values.
template <typename T, int VB>
__device__ __forceinline__ bool all_finite(const T (&v)[VB]) {
    T z = T(0);
#pragma unroll
    for (int c = 0; c < VB; ++c) z += T(0) * v[c];
    return z == T(0);
}

// Fourth word of a raw buffer resource on gfx9: data format 32 bits (a zero
// format makes every load return 0), no stride, no swizzle.
constexpr int kBufferWord3 = 0x00020000;

// A value that is the same in every lane, in scalar registers. What a kernel
// that also writes memory loads through a descriptor stays in vector registers
// otherwise, and so does all that is computed from it.
__device__ __forceinline__ uint32_t uniform(uint32_t v) {
    return uint32_t(__builtin_amdgcn_readfirstlane(int(v)));
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T>
__device__ __forceinline__ T* uniform(T* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<T*>(uint64_t(uniform(uint32_t(v))) | (uint64_t(uniform(uint32_t(v >> 32))) << 32));
}
__device__ __forceinline__ SectorDev uniform(const SectorDev& v) {
    SectorDev s = v;
    s.n_sites = uniform(s.n_sites);
    s.n_up = uniform(s.n_up);
    s.mode = uniform(s.mode);
    s.bw = uniform(s.bw);
    s.dim = uniform(s.dim);
    s.binom = uniform(s.binom);
    s.basis = uniform(s.basis);
    s.clt = uniform(s.clt);
    s.two_s = uniform(s.two_s);
    s.full = uniform(s.full);
    s.lin_hi = uniform(s.lin_hi);
    s.lin_lo = uniform(s.lin_lo);
    s.lin_lo_bits = uniform(s.lin_lo_bits);
    return s;
}

template <typename T>
__device__ __forceinline__ T bond_coef(const BondTable& B, int b) {
    if constexpr (sizeof(T) == 4) return B.coef_f[b];
    else return B.coef_d[b];
}

// The Lanczos epilogue of one row: out = hv_a out - hv_b z with z the row of
// u_{k-1} that y still holds (zero in the first step; ab = [hv_a | hv_b], VB
// each), and the products xt out in FP64.
template <typename T, int VB>
__device__ __forceinline__ void lanczos_epilogue(const T (&xt)[VB], T (&out)[VB], const T* yrow, const T* ab,
                                                 bool first, double (&prod)[VB]) {
    T z[VB];
    if (!first) {
        load_row<T, VB>(yrow, z);
    } else {
#pragma unroll
        for (int c = 0; c < VB; ++c) z[c] = T(0);
    }
#pragma unroll
    for (int c = 0; c < VB; ++c) {
        out[c] = ab[c] * out[c] - ab[VB + c] * z[c];
        prod[c] = double(xt[c]) * double(out[c]);
    }
}

}  // namespace ftlm
