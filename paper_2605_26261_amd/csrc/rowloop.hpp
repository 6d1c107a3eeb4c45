// Row-tile scheduling and deterministic FP64 block reductions shared by the
// persistent row kernels.
#pragma once

#include "kernels.hpp"

namespace ftlm {

// The tiles of kBlock rows owned by block `bid` of a (sub-)grid of G blocks
// in the streaming update kernel: first, first + step, ... below end. With G
// a multiple of 8 and the sub-grid starting at a multiple of 8, block i runs
// on XCD i mod 8 (round-robin dispatch), XCD x gets the x-th contiguous
// eighth of the tiles, and inside a share the XCD's blocks stride.
struct TileSpan {
    uint32_t first, end, step;
};

__device__ __forceinline__ TileSpan tile_span(uint32_t ntiles, uint32_t bid, uint32_t G) {
    if (G >= 8 && (G & 7u) == 0) {
        const uint32_t chunk = (ntiles + 7u) >> 3;
        const uint32_t begin = (bid & 7u) * chunk;
        return {begin + (bid >> 3), begin + chunk < ntiles ? begin + chunk : ntiles, G >> 3};
    }
    return {bid, ntiles, G};
}

// Calls f(tile) for the tiles of tile_span(ntiles, bid, G), in order: the
// update kernel's unstaged widths, so that a block sums the same rows in
// the same order whether its width is staged or not.
template <typename F>
__device__ __forceinline__ void for_each_span_tile(uint32_t ntiles, uint32_t bid, uint32_t G, F&& f) {
    const TileSpan sp = tile_span(ntiles, bid, G);
    for (uint32_t tile = sp.first; tile < sp.end; tile += sp.step) f(tile);
}

// Tiles per XCD super-tile (log2) in the schedule of the kernels that reduce
// (for_each_tile): fixed, because it fixes the order of their sums.
constexpr int kXcdSuperShift = 4;

// Calls f(tile) for the tiles of block `bid` (the gather kernels and the
// start vectors). With G a multiple of 8, the tiles are dealt to the XCDs
// in super-tiles of 2^shift tiles, round-robin:
// super-tile k belongs to XCD k mod 8, and inside its super-tiles an XCD's
// blocks stride by G / 8 tiles. All eight XCDs thus sweep one common front of the
// rows, so the partner rows that miss one XCD's L2 are fetched into the
// shared Infinity Cache once for all of them. Contiguous eighths of the rows
// per XCD were slower at every width (N = 30, CR Lanczos step at 12 columns:
// 38.0 ms against 34.5; super-tiles of 1 to 16 tiles within 1 %, 128 tiles
// 35.7 ms).
template <typename F>
__device__ __forceinline__ void for_each_tile(uint32_t ntiles, uint32_t bid, uint32_t G, int shift, F&& f) {
    if (G >= 8 && (G & 7u) == 0) {
        const uint32_t xcd = bid & 7u, slot = bid >> 3, per = G >> 3;
        const uint32_t supers = (ntiles + (1u << shift) - 1u) >> shift;
        const uint32_t mine = supers > xcd ? (supers - xcd + 7u) / 8u : 0u;  // super-tiles of this XCD
        const uint32_t count = mine << shift;
        for (uint32_t q = slot; q < count; q += per) {
            const uint32_t tile = ((xcd + 8u * (q >> shift)) << shift) + (q & ((1u << shift) - 1u));
            if (tile < ntiles) f(tile);
        }
    } else {
        for (uint32_t tile = bid; tile < ntiles; tile += G) f(tile);
    }
}

// A block's partial sum, stored so that a block on another XCD can read it
// once its ticket count says so: the store goes through to the memory side
// (agent scope), wait_published() waits until it is there, and the reader
// drops what its own caches hold (observe_published) before it reads.
__device__ __forceinline__ void publish(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void wait_published() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's stores are complete
}
__device__ __forceinline__ void observe_published() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent"); }

// One level of wave_fold_columns: lanes l and l ^ off hold partial sums of
// the same columns [lo, hi) in slots [0, SK); the lane with bit `off` clear
// keeps [lo, lo + SN), the other keeps [lo + SN, hi), and each adds the
// partner's partial sum of the columns it keeps to its own (own + partner,
// the order of the xor butterfly). Slots past a lane's columns carry no
// column and are never stored.
template <int SK, int SN, int VB>
__device__ __forceinline__ void fold_level(double (&v)[VB], int off, int lane, int& lo, int& hi) {
    const bool up = (lane & off) != 0;
#pragma unroll
    for (int j = 0; j < SN; ++j) {
        const double keep_lo = v[j];
        const double keep_hi = (SN + j < SK) ? v[SN + j] : 0.0;
        const double recv = __shfl_xor(up ? keep_lo : keep_hi, off, 64);
        v[j] = (up ? keep_hi : keep_lo) + recv;
    }
    const int mid = lo + SN;
    if (up) lo = mid;
    else hi = hi < mid ? hi : mid;
}

// Adds the sums over a wave's 64 lanes of p[0..VB) to dst[0..VB) (LDS), or
// stores them there (ADD false). Each
// column's sum is the one of the xor butterfly over lane offsets 32, 16, ...,
// 1: the same pairs of partial sums are added, in the same order, at every
// level. The columns are reduced by recursive halving, though: at each level
// a lane keeps half of its columns, so VB columns take about VB + 6 exchanges
// instead of 6 VB, and column c ends in the one lane that stores it. Called by
// whole waves; VB <= 64.
template <int VB, bool ADD = true>
__device__ __forceinline__ void wave_fold_columns(const double (&p)[VB], double* dst) {
    constexpr int S1 = (VB + 1) / 2, S2 = (S1 + 1) / 2, S3 = (S2 + 1) / 2;
    constexpr int S4 = (S3 + 1) / 2, S5 = (S4 + 1) / 2, S6 = (S5 + 1) / 2;
    static_assert(S6 == 1, "at most 64 columns");
    const int lane = threadIdx.x & 63;
    double v[VB];
#pragma unroll
    for (int c = 0; c < VB; ++c) v[c] = p[c];
    int lo = 0, hi = VB;
    fold_level<VB, S1>(v, 32, lane, lo, hi);
    fold_level<S1, S2>(v, 16, lane, lo, hi);
    fold_level<S2, S3>(v, 8, lane, lo, hi);
    fold_level<S3, S4>(v, 4, lane, lo, hi);
    fold_level<S4, S5>(v, 2, lane, lo, hi);
    fold_level<S5, S6>(v, 1, lane, lo, hi);
    if (lo < hi) dst[lo] = ADD ? dst[lo] + v[0] : v[0];
}

// Sums v[0..N) over the workgroup in a fixed order (butterfly inside each
// wave, then the waves in order) and stores the total of column c at
// partial[c]. red must hold kWaves * N doubles (LDS).
template <int N>
__device__ __forceinline__ void block_sum(const double (&v)[N], double* red, double* partial, int nc) {
    wave_fold_columns<N, false>(v, red + (threadIdx.x >> 6) * N);
    __syncthreads();
    if (int(threadIdx.x) < nc) {
        double s = 0.0;
        for (int w = 0; w < kWaves; ++w) s += red[w * N + threadIdx.x];
        publish(partial + threadIdx.x, s);
    }
}

// Reports whether this block is the last of the G blocks sharing `ticket` to
// get here (then every published partial is visible to it). Only the partials
// cross XCDs inside a launch, so a block waits for its published stores and
// writes back nothing else; the vectors reach the other XCDs at the end of the
// kernel. With a release fence in its place every block wrote back its XCD's
// L2. That, the fold of all columns at once (block_sum, grid_sum_cols) and one
// lane per chain in the last block took an update launch of 8 FP64 columns
// over 924 rows from 18.4 to 6.2 us, of 16 FP32 columns over 352,716 rows from
// 70 to 22 us, and of 32 over 9.7 million rows from 1272 to 697 us. The last
// block resets the ticket for the next launch.
__device__ __forceinline__ bool last_block(uint32_t* ticket, uint32_t G, int* flag_lds) {
    wait_published();
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t prev = atomicAdd(ticket, 1u);
        *flag_lds = (prev == G - 1) ? 1 : 0;
    }
    __syncthreads();
    const bool last = *flag_lds != 0;
    if (last) observe_published();
    return last;
}

// Called by every block of a persistent launch after its last item: the block
// waits for its published partials and counts itself out. Returns true in the
// last block to get here, with every partial visible to it, after it has
// zeroed the counters for the next launch (every block has stopped taking
// items). No device-scope release: on gfx950 it writes back and invalidates
// the XCD's L2, and the vectors need none before the kernel's end.
__device__ __forceinline__ bool queue_exit(uint32_t* q, uint32_t grid, int* flag_lds) {
    wait_published();
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t done = atomicAdd(q + 8, 1u);
        const bool last = done == grid - 1u;
        if (last)
            for (int i = 0; i < kQueueWords; ++i) atomicExch(q + i, 0u);
        *flag_lds = last ? 1 : 0;
    }
    __syncthreads();
    const bool last = *flag_lds != 0;
    if (last) observe_published();
    return last;
}

// Columns that grid_sum_cols reduces together, and the LDS it needs for them.
template <int VB, int NT = kBlock>
__host__ __device__ constexpr int grid_sum_group() { return VB < 2048 / NT ? VB : 2048 / NT; }
template <int VB, int NT = kBlock>
__host__ __device__ constexpr size_t grid_sum_lds() {
    return sizeof(double) * (NT / 2) * size_t(grid_sum_group<VB, NT>());
}
constexpr size_t kGridSumLds = sizeof(double) * 1024;  // at every width
template <int VB, int NT = kBlock>
__host__ __device__ constexpr int grid_sum_slots() {
    return (VB + grid_sum_group<VB, NT>() - 1) / grid_sum_group<VB, NT>() * grid_sum_group<VB, NT>();
}

// Fixed-order sums over the G block partials of the columns col0 .. col0 +
// nc - 1 (nc <= VB), partials[g * pstride + col]: thread i of NT sums blocks i,
// i + NT, ..., then the block combines the threads as a tree over i, i + NT /
// 2, ..., i + 64, ..., i + 1, so the order depends on G only (and with SPAN = 2
// NT it is that of a block of 2 NT threads, of which one holds two; the threads past
// NT of a larger block only pass the barriers). Up to 2048 / NT
// columns go through the tree together: a few exchanges through LDS, then the
// fold of the first wave, where one column at a time took eight barriers each
// (the Lanczos H.x over 924 rows of 8 FP64 columns: 17.6 -> 11.8 us). tot[c]
// (LDS, grid_sum_slots<VB, NT>() doubles) receives the totals, visible to the
// first wave; red holds grid_sum_lds<VB, NT>() bytes of LDS.
template <int VB, int NT = kBlock, int SPAN = NT>
__device__ __forceinline__ void grid_sum_cols(const double* partials, int G, int pstride, int col0, int nc,
                                              double* red, double* tot) {
    constexpr int W = grid_sum_group<VB, NT>();
    const int tid = int(threadIdx.x);
#pragma unroll 1
    for (int c0 = 0; c0 < nc; c0 += W) {
        double s[W];
#pragma unroll
        for (int c = 0; c < W; ++c) s[c] = 0.0;
        const double* p = partials + col0 + c0;
#pragma unroll 4
        for (int g = tid < NT ? tid : G; g < G; g += SPAN) {
#pragma unroll
            for (int c = 0; c < W; ++c)
                if (c0 + c < nc) s[c] += *gptr(p + size_t(g) * pstride + c);
        }
        if constexpr (SPAN > NT) {
            static_assert(SPAN == 2 * NT, "one or two threads of the order in each");
            double t[W];
#pragma unroll
            for (int c = 0; c < W; ++c) t[c] = 0.0;
#pragma unroll 4
            for (int g = tid + NT; g < G; g += SPAN) {
#pragma unroll
                for (int c = 0; c < W; ++c)
                    if (c0 + c < nc) t[c] += *gptr(p + size_t(g) * pstride + c);
            }
#pragma unroll
            for (int c = 0; c < W; ++c) s[c] += t[c];
        }
        // threads without a partial hold zeros: with 64 blocks or fewer the
        // first wave holds every partial
        for (int half = NT / 2; half >= 64; half >>= 1) {
            if (G <= half) continue;
            __syncthreads();
            if (tid >= half && tid < 2 * half) {
#pragma unroll
                for (int c = 0; c < W; ++c) red[c * half + tid - half] = s[c];
            }
            __syncthreads();
            if (tid < half) {
#pragma unroll
                for (int c = 0; c < W; ++c) s[c] += red[c * half + tid];
            }
        }
        if (tid < 64) {
            double f[W];
#pragma unroll
            for (int c = 0; c < W; ++c) f[c] = s[c];
            wave_fold_columns<W, false>(f, tot + c0);
        }
    }
}

}  // namespace ftlm
