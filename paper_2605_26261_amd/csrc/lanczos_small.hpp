// First half of a Lanczos step on a small sector: more waves to an item and
// more workgroups to a launch than the persistent kernels give it.
#pragma once

#include "hv_impl.hpp"

namespace ftlm {

constexpr int kSmallItems = 256;
constexpr size_t kSmallLds = 144 * 1024;  // most dynamic LDS: the rest of the 160 KB holds the static arrays

// The items of the launch's sector, their slots and their sums are those of
// the persistent kernels. One workgroup runs an item on VB of the launch's
// columns (blockIdx.y): the item's tiles go to NT / 256 groups of four waves at a
// time, each tile's sums per wave are kept apart and added in the tiles' order.
// So neither the threads nor the columns' split change a result. setup(S, c0)
// stages LDS and returns row(t, x, y, ab, first, prod), which writes row t and
// its products.
//
// What bounds it: the latency of one pass over a row (walking its label, then
// gathers in turn). The persistent kernel made four such passes in a row in one
// workgroup per item, on 80 of the 256 CUs for 73,789 rows (icosahedron, s = 1,
// 8 FP64 columns: Lanczos step 93.7 -> 54.8 us; 28,314 rows: 73.7 -> 30.7).
template <typename T, int VB, int NT, typename Setup>
__device__ __forceinline__ void small_lanczos(LanczosLaunch& a, BondTable& B, unsigned char* smem, Setup&& setup) {
    constexpr uint32_t kGroups = NT / kBlock;
    __shared__ int flag;
    __shared__ T ab[2 * VB];
    __shared__ double psum[2][kGroups][kWaves * VB];
    const int lane = threadIdx.x & 63;
    const uint32_t wave = uniform(threadIdx.x >> 6), group = wave / kWaves, quarter = wave % kWaves;
    const SecWork& sw = a.secs[0];
    const uint32_t local = blockIdx.x, items = uniform(sw.items), col0 = a.col0 + blockIdx.y * VB;
    const bool running = uniform(sw.state[1]) != 0;
    if (running) {
        const int step = uniform(sw.state[0]);
        const SectorDev S = uniform(sw.S);
        const T* x = uniform(block_of<T>(a, sw.u[(step - 1) & 1], S.dim));
        T* y = uniform(block_of<T>(a, sw.u[step & 1], S.dim));
        stage_bonds(B, sw.bonds, NT);
        stage_epilogue<T, VB>(ab, sw.chains + col0);
        const auto row = setup(S, col0 - a.block0);
        __syncthreads();
        double sum = 0.0;  // thread t < kWaves VB: wave t / VB, column t % VB
        const uint32_t ntiles = (S.dim + kBlock - 1) / kBlock;
        // the item's n-th tile in for_each_tile's order (ascending)
        auto tile_of = [&](uint32_t n) {
            if (items < 8 || (items & 7u) != 0) return local + n * items;
            const uint32_t q = (local >> 3) + n * (items >> 3);
            return (((local & 7u) + 8u * (q >> kXcdSuperShift)) << kXcdSuperShift) +
                   (q & ((1u << kXcdSuperShift) - 1u));
        };
        int buf = 0;
#pragma unroll 1
        for (uint32_t n = group;; n += kGroups, buf ^= 1) {
            double prod[VB];
#pragma unroll
            for (int c = 0; c < VB; ++c) prod[c] = 0.0;
            const uint64_t t = uint64_t(tile_of(n)) * kBlock + quarter * 64u + uint32_t(lane);
            if (t < S.dim) row(uint32_t(t), x, y, ab, step == 1, prod);
            wave_fold_columns<VB, false>(prod, psum[buf][group] + quarter * VB);
            __syncthreads();
            if (threadIdx.x < kWaves * VB)
                for (uint32_t g = 0; g < kGroups; ++g) sum += psum[buf][g][threadIdx.x];
            if (tile_of(n - group + kGroups) >= ntiles) break;
        }
        __syncthreads();
        double* wsum = psum[0][0];
        if (threadIdx.x < kWaves * VB) wsum[threadIdx.x] = sum;
        __syncthreads();
        if (threadIdx.x < VB) {
            double t = 0.0;
            for (int w = 0; w < kWaves; ++w) t += wsum[w * VB + threadIdx.x];
            publish(sw.partials + size_t(local) * a.ld + col0 + threadIdx.x, t);
        }
    }
    if (queue_exit(a.queue, gridDim.x * gridDim.y, &flag) && running) {
        double* red = reinterpret_cast<double*>(smem);
        if (a.vb == VB) finish_alpha<VB>(sw, a, items, red);
        else if (a.vb == 2) finish_alpha<2>(sw, a, items, red);
        else if (a.vb == 4) finish_alpha<4>(sw, a, items, red);
        else if (a.vb == 8) finish_alpha<8>(sw, a, items, red);
        else finish_alpha<16>(sw, a, items, red);
    }
}

// Spin 1/2, FP64 vectors.
template <typename L, int MODE, int VB, int NT>
__global__ __launch_bounds__(NT) void hv_small_lanczos_kernel(LanczosLaunch a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ BondTable B;
    small_lanczos<double, VB, NT>(a, B, smem, [&](const SectorDev& S, uint32_t col0) {
        const HvLds l = hv_lds_setup<MODE>(smem, S);
        return [=](uint32_t t, const double* x, double* y, const double* ab, bool first, double (&prod)[VB]) {
            walk_row<L, MODE, double, VB>(t, S, B, Binom{l.binom, S.bw}, l.ylds, x, y, a.block_ld, col0, ab, first, prod);
        };
    });
}

// Threads of a workgroup: up to seven items have one tile each and four waves
// do; else sixteen, four tiles at a time.
inline int small_threads(const LanczosLaunch& a) { return a.items < 8 ? kBlock : 4 * kBlock; }

// LDS of a small launch from a workgroup's of kBlock threads, `slabs` bytes of
// which are its waves' own.
inline size_t small_lanczos_lds(const LanczosLaunch& a, size_t lds, size_t slabs) {
    return std::max(lds + slabs * size_t(small_threads(a) / kBlock - 1), kGridSumLds);
}

// One sector with no more items than CUs, while the slabs of its waves fit.
inline bool by_small_lanczos(const LanczosLaunch& a, size_t lds) {
    return a.nsec == 1 && a.items <= kSmallItems && lds <= kSmallLds &&
           (a.vb <= 2 || a.vb == 4 || a.vb == 8 || a.vb == 16);
}

// Columns of a workgroup: 1, 2 or 4, the fewest that keep the workgroups
// within one to a CU (73,789 rows, 80 items, 8 FP64 columns: 55 us with two
// workgroups an item, 89 with four), at most four for the registers.
template <typename F>
hipError_t with_small_shape(const LanczosLaunch& a, F&& g) {
    auto f = [&](auto vb) {
        return small_threads(a) == kBlock ? g(vb, std::integral_constant<int, kBlock>{})
                                          : g(vb, std::integral_constant<int, 4 * kBlock>{});
    };
    int vb = a.vb;
    while (vb > 4 || (vb > 1 && vb % 2 == 0 && a.items * (a.vb / vb) * 2 <= kSmallItems)) vb /= 2;
    if (vb == 1) return f(std::integral_constant<int, 1>{});
    if (vb == 2) return f(std::integral_constant<int, 2>{});
    return f(std::integral_constant<int, 4>{});
}

template <typename K>
hipError_t launch_small_lanczos(K kern, int vb, const LanczosLaunch& a, size_t lds, hipStream_t st) {
    if (!a.queue || a.items <= 0) return hipErrorInvalidValue;  // the queue counters are required
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(unsigned(a.items), unsigned(a.vb / vb)), dim3(unsigned(small_threads(a))), lds, st, a);
    return hipGetLastError();
}

}  // namespace ftlm
