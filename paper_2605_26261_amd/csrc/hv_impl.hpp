// Matrix-free multi-vector H.x kernel (paper Sec. 2, Eq. 12, row-wise gather
// form), templated on label width, indexing mode, element type, vector block
// width and epilogue. Included by hv_f32.hip and hv_f64.hip.
#pragma once

#include <type_traits>

#include "rowio.hpp"
#include "rowloop.hpp"
#include "runs.hpp"

namespace ftlm {

// Accumulates the off-diagonal terms of one row: for each antiparallel bond
// the partner's row of x times J_b / 2; `anti` collects sum J_b / 2 over
// those bonds so the diagonal is sum_b J_b/4 - anti (each antiparallel bond
// turns +J_b/4 into -J_b/4).
// A partner index is in [0, D) by construction; it is clamped there anyway so
// that a defect in the index arithmetic shows up as a parity failure and
// never as an access outside x (by runs: at most a run's length past it, see kRunRows).
template <typename T, int VB, int SG = 2, bool BUF = false>
struct GatherVisitor {
    static_assert(!BUF || VB == 1, "buffer-resource gathers serve single vectors");
    // Column col0 of row 0 of x as bytes, and the row stride in bytes (at
    // most 64 columns of 8 bytes): a partner row's address is then one
    // 32 x 32 -> 64-bit multiply-add.
    const unsigned char* __restrict__ xb;
    uint32_t ldb;
    uint32_t last;  // D - 1
    // BUF: x is one contiguous vector of fewer than 2^32 bytes, read through
    // this buffer resource with 32-bit byte offsets (one shift per partner
    // instead of the clamp and the 64-bit multiply-add); the hardware's range
    // check returns 0 for an offset past the end, so a defect in the index
    // arithmetic still cannot read outside x.
    __amdgpu_buffer_rsrc_t rs;
    __device__ __forceinline__ const T* row(uint32_t i) const {
        return reinterpret_cast<const T*>(xb + uint64_t(i) * ldb);
    }
    const BondTable& B;
    T (&acc)[VB];
    T& anti;
    // row i of x into v (i is clamped into [0, D) on the pointer path)
    __device__ __forceinline__ void gather(uint32_t i, T (&v)[VB]) const {
        if constexpr (BUF) {
            if constexpr (sizeof(T) == 4)
                v[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, int(i << 2), 0, 0));
            else
                v[0] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, int(i << 3), 0, 0));
        } else {
            load_row<T, VB>(row(i < last ? i : last), v);
        }
    }
    __device__ __forceinline__ void flip(int b, uint32_t idx) {
        const T c = bond_coef<T>(B, b);
        T v[VB];
        gather(idx, v);
#pragma unroll
        for (int i = 0; i < VB; ++i) acc[i] += c * v[i];
        anti += c;
    }
    __device__ __forceinline__ void par(int) {}
    // CLT: a group of kGroup consecutive bonds: the rows of the antiparallel
    // ones are loaded together (lanes whose bond is parallel load nothing),
    // then accumulated with weight J_b / 2 or zero. Sizes measured per width
    // (Lanczos step at N = 30): 8 at one column (9.0 -> 8.3 ms against 4),
    // 6 at 8 columns, 3 at 12, 2 from 16 up, 4 elsewhere.
    static constexpr int kGroup = VB == 1 ? 8 : VB == 8 ? 6 : VB == 12 ? 3 : VB >= 16 ? 2 : 4;
    // CR: up to 8 columns, the bonds in slots of kSiteGroup = SG (site_group,
    // per width and epilogue) with two slots in flight (cr_bonds_pairs);
    // wider blocks take one bond at a time (flip /
    // par). Lanczos step at N = 30: one column 15.1 -> 9.6 ms; from 10
    // columns up the two slots were slower (12 columns 36.6 -> 41.5 ms):
    // every lane then loads a full row per bond, parallel lanes included,
    // and the kernel is bound by the traffic, not the latency, of its gathers.
    static constexpr bool kPairs = VB <= 8;
    static constexpr int kSiteGroup = SG;
    // The two slots: rows of x and their weights (J_b / 2 for a flip, else 0).
    // Every lane loads, so the loads are not under a branch and the compiler
    // can wait for exactly the older slot: a lane whose bond is parallel
    // loads row 0 (one cache line shared by all such lanes) under weight zero.
    T slot_a[kSiteGroup][VB], slot_b[kSiteGroup][VB];
    T w_a[kSiteGroup], w_b[kSiteGroup];
    __device__ __forceinline__ void clear_slots() {
#pragma unroll
        for (int g = 0; g < kSiteGroup; ++g) {
            w_a[g] = w_b[g] = T(0);
#pragma unroll
            for (int i = 0; i < VB; ++i) slot_a[g][i] = slot_b[g][i] = T(0);
        }
    }
    // A full slot of kSiteGroup bonds b0, b0 + 1, ...
    __device__ __forceinline__ void load_slot(T (&slot)[kSiteGroup][VB], T (&w)[kSiteGroup], int b0,
                                              const uint32_t (&idx)[kSiteGroup], const bool (&flips)[kSiteGroup]) {
#pragma unroll
        for (int g = 0; g < kSiteGroup; ++g) {
            gather(flips[g] ? idx[g] : 0u, slot[g]);
            const T cb = bond_coef<T>(B, b0 + g);
            w[g] = flips[g] ? cb : T(0);
        }
    }
    __device__ __forceinline__ void add_slot(const T (&slot)[kSiteGroup][VB], const T (&w)[kSiteGroup]) {
#pragma unroll
        for (int g = 0; g < kSiteGroup; ++g) {
#pragma unroll
            for (int i = 0; i < VB; ++i) acc[i] += w[g] * slot[g][i];
            anti += w[g];
        }
    }
    __device__ __forceinline__ void load_slot_a(int b0, const uint32_t (&idx)[kSiteGroup],
                                                const bool (&flips)[kSiteGroup]) {
        load_slot(slot_a, w_a, b0, idx, flips);
    }
    __device__ __forceinline__ void load_slot_b(int b0, const uint32_t (&idx)[kSiteGroup],
                                                const bool (&flips)[kSiteGroup]) {
        load_slot(slot_b, w_b, b0, idx, flips);
    }
    __device__ __forceinline__ void add_slot_a() { add_slot(slot_a, w_a); }
    __device__ __forceinline__ void add_slot_b() { add_slot(slot_b, w_b); }
    __device__ __forceinline__ void group(int b0, const uint32_t (&idx)[kGroup], const bool (&flips)[kGroup]) {
        T v[kGroup][VB];
#pragma unroll
        for (int g = 0; g < kGroup; ++g) {
#pragma unroll
            for (int i = 0; i < VB; ++i) v[g][i] = T(0);
            if (flips[g]) gather(idx[g], v[g]);
        }
#pragma unroll
        for (int g = 0; g < kGroup; ++g) {
            const T cb = bond_coef<T>(B, b0 + g);
            const T c = flips[g] ? cb : T(0);
#pragma unroll
            for (int i = 0; i < VB; ++i) acc[i] += c * v[g][i];
            anti += c;
        }
    }
};

// LDS layout shared by the H.x kernels: FP64 scratch (kBlock doubles), the
// binomial table (CR), then one [site][lane] slab of Y values per wave (CR).
struct HvLds {
    double* red;
    uint32_t* binom;
    uint32_t* ylds;
};

template <int MODE, bool BINOM = (MODE == kModeCr)>
__device__ __forceinline__ HvLds hv_lds_setup(unsigned char* smem, const SectorDev& S) {
    HvLds l;
    l.red = reinterpret_cast<double*>(smem);
    l.binom = reinterpret_cast<uint32_t*>(smem + hv_red_bytes());
    uint32_t* slabs = l.binom + ((S.n_sites * S.bw + 3) & ~3);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    l.ylds = slabs + wave * S.n_sites * 64 + lane;
    if constexpr (BINOM) stage_binomials(l.binom, S.binom, S.n_sites * S.bw);
    return l;
}

// The rows of one block of a (sub-)grid of G blocks: y = H x on rows
// [row0, row0 + nrows), columns [col0, col0 + VB) of [D][ld] blocks. In the
// Lanczos epilogue y holds u_{k-1} on entry (unless `first`) and receives
// w = hv_a (H u_k) - hv_b u_{k-1} per column (ab = [hv_a | hv_b], VB each); the products u_k[t] w[t] are
// folded, tile by tile, into per-wave FP64 sums wsum[wave * VB + c] (LDS).
// Bonds per slot of the two-slot CR pipeline, timed per width at N = 30 (FP32):
//   1-2 columns: three bonds (plain H.x 7.95 -> 7.78 ms at one column, 8.26 ->
//     7.97 at two; Lanczos step 9.74 -> 9.25 ms at two);
//   4 columns: three in the Lanczos step (12.16 -> 11.78 ms), two in the plain
//     H.x (9.6 against 9.7);
//   8 columns: one in the plain H.x (19.9 -> 17.7 ms), two in the Lanczos step
//     (one gave 23.6 ms against 22.0, three 22.5).
// The slot size changes no partner index and no order of accumulation.
constexpr int site_group(int vb, int epi) {
    if (vb <= 2) return 3;
    if (vb == 4) return epi == kEpiLanczos ? 3 : 2;
    if (vb == 8) return epi == kEpiPlain ? 1 : 2;
    return 2;
}

template <typename L, int MODE, typename T, int VB, int EPI, bool BUF = false>
__device__ __forceinline__ void hv_body(const SectorDev& S, const BondTable& B, const HvLds& lds,
                                        const T* __restrict__ x, T* __restrict__ y, uint64_t ld,
                                        uint32_t col0, uint32_t row0, uint32_t nrows, uint32_t bid,
                                        uint32_t G, int shift, const T* ab, bool first, double* wsum) {
    const Binom C{lds.binom, S.bw};
    const int wave = threadIdx.x >> 6;
    const T jsum4 = sizeof(T) == 4 ? T(B.jsum4_f) : T(B.jsum4_d);
    const uint32_t ntiles = (nrows + kBlock - 1) / kBlock;
    for_each_tile(ntiles, bid, G, shift, [&](uint32_t tile) {
        const uint32_t r = tile * kBlock + threadIdx.x;
        const bool valid = r < nrows;
        T xt[VB], out[VB];
        double p[VB];
#pragma unroll
        for (int c = 0; c < VB; ++c) p[c] = 0.0;
        if (valid) {
            const uint32_t t = row0 + r;
            T acc[VB];
#pragma unroll
            for (int c = 0; c < VB; ++c) acc[c] = T(0);
            T anti = T(0);
            GatherVisitor<T, VB, site_group(VB, EPI), BUF> vis{
                reinterpret_cast<const unsigned char*>(x + col0), uint32_t(ld * sizeof(T)), S.dim - 1,
                __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(x), 0, BUF ? int(uint64_t(S.dim) * sizeof(T)) : 0,
                                                  kBufferWord3),
                B, acc, anti};
            visit_row<L, MODE>(t, S.n_up, B, C, S.basis, table_map<MODE>(S), lds.ylds, vis);
            load_row<T, VB>(x + uint64_t(t) * ld + col0, xt);
            if constexpr (EPI == kEpiPlain && MODE == kModeCr && VB <= 8) {
                // the two slots weigh row 0 by zero for a bond that does not
                // flip: an infinity or a NaN there makes the sum a NaN, and the
                // row is walked once more, loading its own terms only
                if (!all_finite<T, VB>(acc)) {
#pragma unroll
                    for (int c = 0; c < VB; ++c) acc[c] = T(0);
                    anti = T(0);
                    cr_bonds<L, false>(t, L(0), S.n_up, B, C, lds.ylds, vis);
                }
            }
            const T diag = jsum4 - anti;
#pragma unroll
            for (int c = 0; c < VB; ++c) out[c] = diag * xt[c] + acc[c];
            T* yrow = y + uint64_t(r) * ld + col0;
            if constexpr (EPI == kEpiLanczos) lanczos_epilogue<T, VB>(xt, out, yrow, ab, first, p);
            store_row<T, VB>(yrow, out);
        }
        if constexpr (EPI == kEpiLanczos) {
            // every lane takes part; rows past the end add 0
            wave_fold_columns<VB>(p, wsum + wave * VB);
        }
    });
}

// Every H.x kernel reads its bond table from a copy in a static LDS object:
// the row loop's bond reads become broadcast LDS reads, which lets the
// compiler keep several partner rows in flight per thread (read from kernel
// arguments or through a generic pointer, the table costs scalar or flat
// loads whose waits serialise the gathers). Visible after the caller's next
// barrier.
__device__ __forceinline__ void stage_bonds(BondTable& dst, const BondTable* src, int threads = kBlock) {
    uint32_t* d = reinterpret_cast<uint32_t*>(&dst);
    const uint32_t* w = reinterpret_cast<const uint32_t*>(src);
    for (int i = threadIdx.x; i < int(sizeof(BondTable) / 4); i += threads) d[i] = *gptr(w + i);
}

template <typename L, int MODE, typename T, int VB, bool BUF = false>
__global__ __launch_bounds__(kBlock) void hv_kernel(SectorDev S, BondTable B, HvLaunch h) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ BondTable Bs;
    stage_bonds(Bs, &B);
    const HvLds lds = hv_lds_setup<MODE>(smem, S);
    __syncthreads();
    hv_body<L, MODE, T, VB, kEpiPlain, BUF>(S, Bs, lds, static_cast<const T*>(h.x), static_cast<T*>(h.y), h.ld, h.col0,
                                        h.row0, h.nrows, blockIdx.x, gridDim.x, h.super_shift, nullptr, false, nullptr);
}

// How the run kernel takes rows of a given size: rows a lane, sites of the low
// part, rows a wave takes at a time at most, and blocks at most. Icosidodecahedron,
// N = 30: 4-byte rows 3.0 ms with 4 rows a lane and 14 sites (2 rows 3.6, 1 row
// 4.8; 13 sites 3.1-3.3), 8-byte rows 5.1 (2 rows, 13 sites; 14 sites 5.4-6.0),
// 16-byte rows 7.3 (12 and 14 sites 7.5; one row a lane 8.1), 32-byte rows
// 14.4 (12 sites, 64 rows a wave; 128 rows 15.2). Narrow rows spread over 8192
// blocks, whose rank tables are staged once for several tiles; for wider ones
// a block takes one tile, see walk_schedule.
struct RunShape {
    int lane_rows, low_bits;
    uint32_t chunk, blocks;
};
constexpr RunShape run_shape(size_t row_bytes) {
    return row_bytes <= 4    ? RunShape{4, 14, 1024, 8192}
           : row_bytes <= 8  ? RunShape{2, 13, 512, 1u << 30}
           : row_bytes <= 16 ? RunShape{2, 13, 256, 1u << 30}
                             : RunShape{1, 12, 64, 1u << 30};
}
constexpr int kRunGroup = 2;  // bonds a slot: 4 or 8 gave 3.3 and 4.1 ms for 4-byte rows, 4 8.1 for 16-byte rows

// The plain H.x by runs: every wave takes `chunk` consecutive rows at a time
// (runs.hpp), four waves a block, the blocks in for_each_tile's order.
//
// What bounds it. One FP32 vector at N = 30: 3.0 ms against 7.4 for the
// row-by-row kernel, whose 1400 VALU instructions per 64 rows index every
// row's partners on their own; by runs the high sites' share is computed once
// per run and a partner costs a mask, a count, one LDS read and a
// multiply-add, about 500 in all. From 16-byte rows on the lines missed in L2
// bound it (that path gives 7 TB/s, whether the Infinity Cache holds the line
// or not): four FP32 columns 9.4 -> 7.3 ms, eight 17.7 -> 14.4.
//
// Short runs lie together, in sectors with fewer up than down spins at the end,
// and their waves take longest: a launch with a block for every tile begins with
// them (25 sites, 11 up, two FP32 columns: 185 us in ascending order, 142 this way
// and with 14 up; where a block takes several tiles, 29 sites, 10 up, one column:
// 640 and 666).
template <typename L, typename T, int VB>
__global__ __launch_bounds__(kBlock) void hv_runs_kernel(SectorDev S, BondTable B, HvLaunch h) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ BondTable Bs;
    stage_bonds(Bs, &B);
    const int low_bits = h.low_bits;
    uint32_t* low = reinterpret_cast<uint32_t*>(smem);
    const uint32_t* src = reinterpret_cast<const uint32_t*>(kLow.rank);
    for (int i = threadIdx.x; i < (1 << low_bits) / 2; i += kBlock) low[i] = *gptr(src + i);
    uint32_t* binom = low + (1 << low_bits) / 2;
    stage_binomials(binom, S.binom, S.n_sites * S.bw);
    const Binom C{binom, S.bw};
    const uint32_t wave = uint32_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)));
    const uint32_t block_rows = kWaves * h.chunk;
    const uint32_t ntiles = uint32_t((uint64_t(h.nrows) + block_rows - 1) / block_rows);
    for_each_tile(ntiles, blockIdx.x, gridDim.x, h.super_shift, [&](uint32_t i) {
        const uint32_t tile = (ntiles & h.flip) + (i ^ h.flip);  // i, or ntiles - 1 - i
        const uint64_t r0 = uint64_t(tile) * block_rows + uint64_t(wave) * h.chunk;
        if (r0 >= h.nrows) return;
        const uint32_t n = h.nrows - uint32_t(r0) < h.chunk ? h.nrows - uint32_t(r0) : h.chunk;
        const uint32_t pos = h.row0 + uint32_t(r0);
        run_rows<L, T, VB, run_shape(VB * sizeof(T)).lane_rows, kRunGroup>(S, Bs, smem, C, low_bits,
                                                                  static_cast<const T*>(h.x), static_cast<T*>(h.y),
                                                                  h.ld, h.col0, h.row0, pos, pos + n);
    });
}

// The epilogue scalars [hv_a | hv_b] of columns [col0, col0 + VB), in the
// vector precision, into LDS; visible after the caller's next barrier.
template <typename T, int VB>
__device__ __forceinline__ void stage_epilogue(T* ab, const Chain* chains) {
    if (threadIdx.x < VB) {
        const Chain* ch = chains + threadIdx.x;
        ab[threadIdx.x] = sizeof(T) == 4 ? T(ch->hv_a_f) : T(ch->hv_a_d);
        ab[VB + threadIdx.x] = sizeof(T) == 4 ? T(ch->hv_b_f) : T(ch->hv_b_d);
    }
}

// Row t of a Lanczos step by one lane: w = hv_a (H u_k) - hv_b u_{k-1} and the
// products u_k w. `ylds` is the lane's own [site] column of Y values (ranking).
template <typename L, int MODE, typename T, int VB>
__device__ __forceinline__ void walk_row(uint32_t t, const SectorDev& S, const BondTable& B, Binom C, uint32_t* ylds,
                                         const T* __restrict__ x, T* __restrict__ y, uint64_t ld, uint32_t col0,
                                         const T* ab, bool first, double (&prod)[VB]) {
    T acc[VB], xt[VB], out[VB];
#pragma unroll
    for (int c = 0; c < VB; ++c) acc[c] = T(0);
    T anti = T(0);
    GatherVisitor<T, VB, site_group(VB, kEpiLanczos)> vis{
        reinterpret_cast<const unsigned char*>(x + col0), uint32_t(ld * sizeof(T)), S.dim - 1,
        __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(x), 0, 0, kBufferWord3), B, acc, anti};
    visit_row<L, MODE>(t, S.n_up, B, C, S.basis, table_map<MODE>(S), ylds, vis);
    load_row<T, VB>(x + uint64_t(t) * ld + col0, xt);
    const T diag = (sizeof(T) == 4 ? T(B.jsum4_f) : T(B.jsum4_d)) - anti;
#pragma unroll
    for (int c = 0; c < VB; ++c) out[c] = diag * xt[c] + acc[c];
    T* yrow = y + uint64_t(t) * ld + col0;
    lanczos_epilogue<T, VB>(xt, out, yrow, ab, first, prod);
    store_row<T, VB>(yrow, out);
}

// The block's FP64 partials of <u_k, w> for its VB columns (wsum: one row of
// VB per wave) into its slot of the sector's partials.
template <int VB>
__device__ __forceinline__ void store_partials(const SecWork& sw, const LanczosLaunch& a, const double* wsum,
                                               uint32_t slot) {
    __syncthreads();
    if (threadIdx.x < VB) {
        double t = 0.0;
        for (int w = 0; w < kWaves; ++w) t += wsum[w * VB + threadIdx.x];
        publish(sw.partials + size_t(slot) * a.ld + a.col0 + threadIdx.x, t);
    }
}

// alpha_k of the launch's columns of one sector from its n partial slots, one
// thread per column.
template <int VB, int NT = kBlock, int SPAN = NT>
__device__ __forceinline__ void finish_alpha(const SecWork& sw, const LanczosLaunch& a, uint32_t n, double* red) {
    __shared__ double tot[grid_sum_slots<VB, NT>()];
    grid_sum_cols<VB, NT, SPAN>(sw.partials, int(n), int(a.ld), int(a.col0), VB, red, tot);
    if (threadIdx.x < VB) {
        chain_set_alpha(&sw.chains[a.col0 + threadIdx.x], tot[threadIdx.x]);
    }
}

// First half of Lanczos step k over every sector of the launch (one sector,
// all sectors of a plan, or a server round): w = H q_k - beta_{k-1} q_{k-1}
// and the FP64 partials of <u_k, w>, summed in slot order into alpha_k (and
// the update coefficient). A sector whose chains have all stopped is skipped.
//
// The grid is persistent, sized to the resident workgroups: each workgroup
// takes (sector, item) pairs from its XCD's counter (queue_item) and runs
// them one after the other, and each item stores its partials in its own
// slot. The last workgroup to leave (queue_exit) sums every sector's slots. Which
// workgroup ran an item changes nothing: the tiles of an item, its partial
// slot and the summation order depend on the sector's dimension only.
template <typename L, int MODE, typename T, int VB>
__global__ __launch_bounds__(kBlock) void hv_lanczos_kernel(LanczosLaunch a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int flag;
    __shared__ uint32_t next;
    __shared__ BondTable B;
    __shared__ T ab[2 * VB];
    const SecWork* secs = a.secs;
    const uint32_t xcd = blockIdx.x & 7u;
    for (;;) {
        if (threadIdx.x == 0) next = atomicAdd(a.queue + xcd, 1u);
        __syncthreads();
        uint32_t local = 0;
        const int s = uniform(queue_item(secs, a.nsec, xcd, next, &local));
        __syncthreads();  // every thread has read `next`
        if (s < 0) break;
        local = uniform(local);
        const SecWork& sw = secs[s];
        if (uniform(sw.state[1]) == 0) continue;
        const int step = uniform(sw.state[0]);
        const SectorDev S = uniform(sw.S);
        stage_bonds(B, sw.bonds);
        stage_epilogue<T, VB>(ab, sw.chains + a.col0);
        const HvLds lds = hv_lds_setup<MODE>(smem, S);
        double* wsum = lds.red;
        for (int i = threadIdx.x; i < kWaves * VB; i += kBlock) wsum[i] = 0.0;
        __syncthreads();
        const T* x = uniform(block_of<T>(a, sw.u[(step - 1) & 1], S.dim));
        T* y = uniform(block_of<T>(a, sw.u[step & 1], S.dim));
        hv_body<L, MODE, T, VB, kEpiLanczos>(S, B, lds, x, y, a.block_ld, a.col0 - a.block0, 0, S.dim, local, uniform(sw.items),
                                             kXcdSuperShift, ab, step == 1, wsum);
        store_partials<VB>(sw, a, wsum, local);
        __syncthreads();  // LDS (bonds, scalars, tables) is restaged by the next item
    }
    if (queue_exit(a.queue, gridDim.x, &flag)) {
        double* red = reinterpret_cast<double*>(smem);
        for (int s = 0; s < a.nsec; ++s)
            if (uniform(secs[s].state[1]) != 0) finish_alpha<VB>(secs[s], a, secs[s].items, red);
    }
}

// Dynamic LDS of the plain H.x at 20 and more FP32 columns: enough that three
// workgroups fill a CU's 160 KB. With more rows in flight the partner rows are
// evicted before their reuse (N = 30, 20 columns: 40.5 -> 38.9 ms; two
// workgroups 44.9). Narrower blocks keep the register-limited occupancy (8
// columns: 15.9 against 18.1 ms with the floor, 16: 31.3 against 33.6).
// A product of 32 columns over few rows has no such choice of rows in flight: up to
// 768 tiles all are resident at once, three to a CU, without a floor (722 tiles 78.9
// us, 82.2 with two workgroups, but 20 columns 44.9 and 42.9); up to 1024 it would be
// four (33 sites, 28 up, 928 tiles 126 us, 104 with two; 64 columns, 795 tiles 221
// and 184). Rows of more than 32 columns that are not whole lines take several
// launches, each of which fetches lines of its neighbours: two workgroups (52
// columns, 705,432 rows 666 us with three, 609 with two; 64 columns 526 and 565).
inline bool two_to_a_cu(const HvLaunch& h) {
    return h.dtype == 0 && h.vb >= 20 && h.ld % 32 != 0 && (h.ld > 32 || h.nrows <= (1u << 18));
}
template <typename T, int VB>
size_t hv_plain_lds_floor(const HvLaunch& h) {
    if (sizeof(T) != 4 || VB < 20) return 0;
    if (two_to_a_cu(h)) return size_t(72) * 1024;
    const uint64_t tiles = (uint64_t(h.nrows) + kBlock - 1) / kBlock;
    return tiles <= 768 ? 0 : size_t(tiles <= 1024 ? 72 : 48) * 1024;
}

template <typename L, int MODE, typename T, int VB, bool BUF = false>
hipError_t launch_hv_one(const SectorDev& s, const BondTable& B, const HvLaunch& h, hipStream_t st) {
    const size_t need = hv_lds_bytes(s), floor = hv_plain_lds_floor<T, VB>(h);
    const size_t lds = need > floor ? need : floor;
    auto kern = hv_kernel<L, MODE, T, VB, BUF>;
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(unsigned(h.grid)), dim3(kBlock), lds, st, s, B, h);
    return hipGetLastError();
}

// Grid of a persistent launch: the resident workgroups of the kernel at this
// LDS size (a multiple of 8, so every XCD gets the same number), capped at
// the number of work items.
hipError_t persistent_grid(const void* kern, int threads, size_t lds, int items, int* grid);

template <typename L, int MODE, typename T, int VB>
hipError_t launch_lanczos_one(const LanczosLaunch& a, size_t lds, hipStream_t st) {
    auto kern = hv_lanczos_kernel<L, MODE, T, VB>;
    if (lds < kGridSumLds) lds = kGridSumLds;  // the final sums reuse the block's LDS
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
        if (e != hipSuccess) return e;
    }
    if (!a.queue || a.items <= 0) return hipErrorInvalidValue;  // the queue counters are required
    int grid = 0;
    hipError_t e = persistent_grid(reinterpret_cast<const void*>(kern), kBlock, lds, a.items, &grid);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(unsigned(grid)), dim3(kBlock), lds, st, a);
    return hipGetLastError();
}

// Dispatch over the vector-block width VB (columns per launch).
template <typename T, typename F>
hipError_t with_vb(int vb, F&& f) {
    switch (vb) {
        case 1: return f(std::integral_constant<int, 1>{});
        case 2: return f(std::integral_constant<int, 2>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 8: return f(std::integral_constant<int, 8>{});
        case 16: return f(std::integral_constant<int, 16>{});
        case 10:
            if constexpr (sizeof(T) == 4) return f(std::integral_constant<int, 10>{});
            else return hipErrorInvalidValue;
        case 12:
            if constexpr (sizeof(T) == 4) return f(std::integral_constant<int, 12>{});
            else return hipErrorInvalidValue;
        case 20:
            if constexpr (sizeof(T) == 4) return f(std::integral_constant<int, 20>{});
            else return hipErrorInvalidValue;
        case 32:
            if constexpr (sizeof(T) == 4) return f(std::integral_constant<int, 32>{});
            else return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

// Dispatch over label width and indexing mode.
template <typename F>
hipError_t with_mode(int mode, int n_sites, F&& f) {
    if (mode == kModeClt) return f(uint32_t{}, std::integral_constant<int, kModeClt>{});
    if (mode == kModeFull) return f(uint32_t{}, std::integral_constant<int, kModeFull>{});
    if (mode == kModeLin) return f(uint32_t{}, std::integral_constant<int, kModeLin>{});
    if (n_sites > 32) return f(uint64_t{}, std::integral_constant<int, kModeCr>{});
    return f(uint32_t{}, std::integral_constant<int, kModeCr>{});
}

// Tiles per XCD super-tile (log2) of a plain H.x over `ntiles` tiles: 64 tiles
// (24-site square lattice, 8 columns: 363 us with 16, 342 with 64, 375 with
// 256; N = 30 within 0.3 %) or 2^most, fewer where there would be less than
// `least` super-tiles.
inline int plain_super_shift(uint64_t ntiles, int most, uint64_t least = 128) {
    int s = most;
    while (s > 0 && (ntiles >> s) < least) --s;
    return s;
}

// The same for a grid with a block for every tile: the largest with which no
// block of an XCD takes a second tile while another has none (692 tiles, one FP32
// column: 12.1 us with single tiles, 19.7 with 2, 4, 8 or 16).
inline int single_tile_shift(uint64_t ntiles, int most) {
    int s = most;
    for (; s > 0; --s) {
        const uint64_t full = ntiles >> s, part = ntiles & ((uint64_t(1) << s) - 1);
        const uint64_t xcd0 = full % 8 ? (full / 8 + 1) << s : (full / 8 << s) + part;
        if (xcd0 <= (ntiles + 7) / 8) break;
    }
    return s;
}

// Runs of a sector whose low part has `low_bits` sites, as a double.
inline double run_count(int n_sites, int n_up, int low_bits) {
    double runs = 0.0, c = 1.0;  // c = C(n_sites - low_bits, a)
    const int nh = n_sites - low_bits;
    for (int a = 0; a <= nh && a <= n_up; ++a) {
        if (n_up - a <= low_bits) runs += c;
        c = c * double(nh - a) / double(a + 1);
    }
    return runs;
}

// Whether a product over all rows of a sector, `row_bytes` each, goes by runs.
// Below about a million rows the row-by-row kernel's shorter start wins (N = 22,
// one FP32 vector: 30 against 40 us; N = 23: 55 against 49; N = 24: 110 against 79;
// 8-byte rows a doubling higher). 16-byte rows have the line at `least16` million
// of them: 32 for FP32 products (20.1 M rows 1029 us row by row, 1064 by runs; 40.1
// M 1990 and 1840), 8 for FP64 ones (5.2 M 217 and 224; 10.4 M 542 and 509), 4 for
// the Lanczos step of FP32 vectors (10.4 M, with its update, 717 and 637). A run costs
// about two passes of a wave whatever its length, so there must be rows to
// each: sectors near half filling have 400 runs per million rows with 14 low
// sites and twice as many per site less. With three times as many, 13 million
// rows still gain (28 sites, 18 up, 8-byte rows 558 -> 532 us), but not one FP32
// vector of a sector with a table (345 -> 441; the third of three, whose lines are
// wider, does: 1134 -> 991 in all), and 3 million lose (26 sites, 17 up: 156
// -> 290 us); above 32 sites, where the row-by-row
// kernel walks 64-bit labels, ten times as many still pay (34 sites, 10 up:
// 10.7 -> 7.2 ms; five with 16-byte rows). A Lanczos step of two or four FP32 columns,
// whose row-by-row kernel keeps the rows in flight together, has `most8` and `most16`
// = 6 and 2 (two: 34 sites, 10 up, 8.0 times as many, 9.1 ms row by row, 12.3 by runs,
// 35, 11 up, 5.9 times 36.0 and 30.1; four: 34, 11 up, 4.9 times 24.0 and 30.3, 33,
// 14 up, 1.25 times 68.1 and 65.6). 32-byte rows are bound by the lines they miss either way
// and gain only in the largest sectors (N = 30: 15.9 -> 14.4 ms, N = 28 equal);
// wider rows do not (16 FP32 columns: 31.2 against 32.2 ms).
inline bool by_runs(const SectorDev& s, size_t row_bytes, double least16, bool part = false, double most8 = 10.0,
                    double most16 = 5.0) {
    if (row_bytes > 32) return false;
    const RunShape shape = run_shape(row_bytes);
    if (s.n_sites <= shape.low_bits) return false;
    const bool table = s.mode == kModeClt || s.mode == kModeLin;
    const double dim = double(s.dim);
    const double least = row_bytes <= 4 ? (table ? 4.0 : 1.25) : row_bytes <= 8 ? 2.0 : row_bytes <= 16 ? least16 : 64.0;
    if (dim < least * 1048576.0) return false;
    const double unit = double(1u << (14 - shape.low_bits)) * 500e-6 * dim;  // 500 per million rows at 14 sites
    const double runs = run_count(s.n_sites, s.n_up, shape.low_bits);
    if (runs <= unit) return true;
    if (row_bytes > 16) return false;
    if (s.n_sites > 32 && dim >= 67108864.0) return runs <= (row_bytes <= 4 ? 10.0 : row_bytes <= 8 ? most8 : most16) * unit;
    return row_bytes <= 8 && dim >= 12582912.0 && runs <= (table && row_bytes <= 4 && !part ? 2.0 : 4.0) * unit;
}

// Pascal's triangle for the host's counts (C(64, 32) < 2^63).
struct Choose {
    uint64_t c[kMaxSites + 1][kMaxSites + 1];
    constexpr Choose() : c{} {
        for (int n = 0; n <= kMaxSites; ++n) {
            c[n][0] = 1;
            for (int k = 1; k <= n; ++k) c[n][k] = c[n - 1][k - 1] + (k < n ? c[n - 1][k] : 0);
        }
    }
};
inline constexpr Choose kChoose{};

// Runs that begin before the one of sector row `row`.
inline uint64_t runs_before(int n_sites, int n_up, int low_bits, uint64_t row) {
    uint64_t runs = 0;
    int A = n_up;  // up spins among the sites 0 .. p
    for (int p = n_sites - 1; p >= low_bits && A > 0; --p) {
        const uint64_t rows = A <= p ? kChoose.c[p][A] : 0;  // with site p down
        if (row < rows) continue;
        const int nh = p - low_bits;
        for (int a = A > low_bits ? A - low_bits : 0; a <= nh && a <= A; ++a) runs += kChoose.c[nh][a];
        row -= rows;
        --A;
    }
    return runs;
}

// Whether a product over a share of a sector's rows goes by runs: where one over
// all rows does, if the share has enough rows and enough of them to a run. The
// runs are counted, as a sector's first and last rows have many short ones. One
// FP32 vector, microseconds by runs and row by row: N = 30, 2^16 rows 23 and 14,
// 2^20 from the middle 55 and 62, from the end 117 and 62, 2^22 from the middle
// 115 and 203, from the end 200 and 204; N = 34, 11 up, 64-bit labels, 2^20 from
// the beginning 46 and 90, from the middle 199 and 90, 2^23 577 and 696. A row is
// dearer with wider vectors or 64-bit labels, a run costs about the same.
inline bool share_by_runs(const SectorDev& s, size_t row_bytes, bool f64, const HvLaunch& h) {
    const uint32_t row0 = h.row0, nrows = h.nrows;
    if (!by_runs(s, row_bytes, f64 ? 8.0 : 32.0, h.ld > uint64_t(h.vb))) return false;
    if (nrows == s.dim) return true;
    const int low = run_shape(row_bytes).low_bits;
    const uint64_t runs = runs_before(s.n_sites, s.n_up, low, uint64_t(row0) + nrows - 1) -
                          runs_before(s.n_sites, s.n_up, low, row0) + 1;
    const bool table = s.mode == kModeClt || s.mode == kModeLin;
    double least, per_run;  // rows
    if (row_bytes <= 4) least = table ? 1.5 : 1.0, per_run = table ? 1200.0 : 700.0;
    else if (row_bytes <= 8) least = table ? 1.0 : 1.25, per_run = table ? 650.0 : 500.0;
    else least = row_bytes <= 16 ? 3.0 : 1.0, per_run = 250.0;
    if (s.n_sites > 32) least *= 2.0, per_run *= 0.35;
    return double(nrows) >= least * 1048576.0 + per_run * double(runs);
}

template <typename L, typename T, int VB>
hipError_t launch_hv_runs(const SectorDev& s, const BondTable& B, HvLaunch h, hipStream_t st) {
    constexpr RunShape shape = run_shape(VB * sizeof(T));
    constexpr uint32_t kStep = 64u * uint32_t(shape.lane_rows);
    h.low_bits = shape.low_bits;
    // Fewer rows a wave where 8192 waves would not all get some, and where
    // short runs lie together and a wave with many of them would end last (28
    // sites, 18 up, one FP32 vector: 1024 rows a wave 570 us, 256 rows 413).
    uint32_t steps = h.nrows / (8192u * kStep);
    steps = steps < 1 ? 1 : steps > shape.chunk / kStep ? shape.chunk / kStep : steps;
    if (run_count(s.n_sites, s.n_up, shape.low_bits) > 600e-6 * double(1u << (14 - shape.low_bits)) * double(s.dim))
        steps = steps < 256u / kStep ? steps : 256u / kStep;
    h.chunk = steps * kStep;
    const uint64_t blocks = (uint64_t(h.nrows) + kWaves * h.chunk - 1) / (uint64_t(kWaves) * h.chunk);
    h.grid = int(blocks < 8 ? blocks : blocks < shape.blocks ? (blocks + 7) & ~uint64_t(7) : shape.blocks);
    h.super_shift = plain_super_shift(blocks, 6);
    h.flip = 2 * s.n_up < s.n_sites && blocks <= shape.blocks ? ~0u : 0u;
    const size_t lds = (size_t(2) << h.low_bits) + size_t(s.n_sites) * size_t(s.bw) * 4;
    hipLaunchKernelGGL((hv_runs_kernel<L, T, VB>), dim3(unsigned(h.grid)), dim3(kBlock), lds, st, s, B, h);
    return hipGetLastError();
}

// The index map that the row-by-row kernel uses in a sector that holds one:
// its own while latency counts and for rows of up to 8 bytes, where a lookup
// is shorter than the ranking walk (N = 18, 8 FP32 columns: compressed table 20
// us, ranking 26; N = 23, one column: 40 against 55), the ranking from 2^18
// rows on for wider rows, where the table's loads come on top of the rows' (N
// = 26, 17 up, 8 columns: 308 against 271 us; N = 30: 22.4 against 15.9 ms) and
// in place of the full table at any width (N = 26, 17 up, one column: 301
// against 146 us). 16 FP64 columns keep the map at any size: the ranking takes
// such rows bond by bond, the maps two at a time (N = 24: table 1034, ranking 1250
// us; N = 27 9.7 and 12.4 ms).
inline int product_map(const SectorDev& s, size_t row_bytes, bool f64, uint32_t nrows) {
    const bool rank = nrows >= (1u << 18) && (row_bytes > 8 || s.mode == kModeFull) && !(f64 && row_bytes >= 128);
    return rank ? kModeCr : s.mode;
}

// Blocks of the row-by-row kernel and its super-tiles. Rows of up to 16 bytes: a
// persistent grid of at most 2048 (latency-bound; one block per tile, whose tables
// are staged each time, gave 8.0 against 7.4 ms at one column). Wider rows are
// bound by the lines they miss in L2, and a block takes one tile: blocks are
// dispatched in order, so the rows in flight stay one compact front, where the
// blocks of a persistent grid drift apart and share fewer partner rows. N = 30,
// FP32: 8 columns 17.7 -> 15.9 ms, 12 28.9 -> 23.7, 16 42.0 -> 31.2, 20 55.4 ->
// 38.9, 4 FP64 columns 19.5 -> 14.8.
// Up to `few_tiles` most blocks of a persistent grid take one tile or a few and
// have no time to drift: it saves the staging. While the latency of a tile bounds
// them, no block takes two tiles (single_tile_shift): up to 1280 tiles, 2048 for
// narrow rows whose partners come from a table, 512 for rows that are a part of a
// wider one and with two workgroups to a CU, which wait for lines (1378 tiles, one
// FP32 column, table 11.5 us with single tiles, 14.0 with 8, ranking 18.3 with
// either; 722 tiles, 52 columns 177 and 151). Beyond, eight super-tiles to an XCD do,
// of up to 32 tiles. Microseconds, one tile a block (super-tiles as for large
// sectors) and this: 1378 tiles, 8, 16 and 20 FP32 columns 30.0, 63.9, 66.2 and
// 28.1, 60.4, 61.7; 2755 tiles, 8, 10, 16 and 32 54.0, 87.7, 122.6, 275 and 49.9,
// 77.9, 113.9, 262; 10,564 tiles, 8 columns 178 and 198.
inline void walk_schedule(size_t row_bytes, uint32_t few_tiles, bool table, HvLaunch& h) {
    const uint64_t ntiles = (uint64_t(h.nrows) + kBlock - 1) / kBlock;
    const bool narrow = row_bytes <= 16;
    if (!narrow && ntiles >= few_tiles) {
        h.grid = int(capped_grid(h.nrows, 1u << 30));
        h.super_shift = plain_super_shift(ntiles, 6);
        return;
    }
    const uint64_t stride = h.ld * (h.dtype == 0 ? 4 : 8);
    const bool part = (stride > row_bytes && stride > 64) || two_to_a_cu(h);
    h.grid = int(rows_grid(h.nrows));
    h.super_shift = ntiles <= (part ? 512 : narrow && table ? 2048 : 1280) ? single_tile_shift(ntiles, 4)
                    : part && ntiles <= 1024                               ? plain_super_shift(ntiles, 4, 40)
                    : narrow ? plain_super_shift(ntiles, 4, part ? 64 : 128)
                             : plain_super_shift(ntiles, 5, 64);
}

// Tiles from which on wide rows take one tile a block. FP32 rows of up to 80 bytes
// and 64-bit labels: 8192 (5282 tiles, 8, 10 and 20 FP32 columns 87.8, 136.7 and
// 251.8 us one tile a block, 84.7, 129.2 and 228.4 on the persistent grid; 48 sites,
// 6689 tiles, 4 FP64 columns 300 and 284); else 4096 (32 FP32 columns 471 and 499,
// 4 FP64 columns 80.7 and 81.7). FP32 rows of up to 40 bytes in sectors with few up,
// or down, spins, which miss fewer lines: 16384 (28 sites, 20 up, 12,142 tiles, 8
// columns 237 and 213).
inline bool few_flips(int n_up, int most) { return 20 * (n_up < most - n_up ? n_up : most - n_up) < 7 * most; }
inline uint32_t few_tiles(const SectorDev& s, size_t row_bytes, bool f32) {
    if (f32 && row_bytes <= 40 && few_flips(s.n_up, s.n_sites)) return 16384;
    return s.n_sites > 32 || (f32 && row_bytes <= 80) ? 8192 : 4096;
}

// A single contiguous vector of fewer than 2^32 bytes takes the
// buffer-resource gathers (GatherVisitor, BUF) with CR and the compressed
// table. N = 30, one FP32 vector: CR 7.77 -> 7.37 ms, CLT 6.06 -> 5.90; FP64
// CR 8.33 -> 7.96. Lin's tables were 2 % slower and the full table
// unchanged, so they keep the pointer form; reading the compressed table
// through a buffer as well changed nothing.
template <typename T>
hipError_t launch_hv_typed(const SectorDev& s, const BondTable& B, const HvLaunch& h0, hipStream_t st) {
    const size_t row_bytes = size_t(h0.vb) * sizeof(T);
    HvLaunch h = h0;
    if (share_by_runs(s, row_bytes, sizeof(T) == 8, h)) {
        auto go = [&](auto vb) {
            constexpr int VB = decltype(vb)::value;
            return s.n_sites > 32 ? launch_hv_runs<uint64_t, T, VB>(s, B, h, st)
                                  : launch_hv_runs<uint32_t, T, VB>(s, B, h, st);
        };
        if (h.vb == 1) return go(std::integral_constant<int, 1>{});
        if (h.vb == 2) return go(std::integral_constant<int, 2>{});
        if (h.vb == 4) return go(std::integral_constant<int, 4>{});
        if constexpr (sizeof(T) == 4)
            if (h.vb == 8) return go(std::integral_constant<int, 8>{});
    }
    const int mode = product_map(s, row_bytes, sizeof(T) == 8, h.nrows);
    walk_schedule(row_bytes, few_tiles(s, row_bytes, sizeof(T) == 4), mode != kModeCr, h);
    const bool buf = h.vb == 1 && h.ld == 1 && h.col0 == 0 && uint64_t(s.dim) * sizeof(T) < (uint64_t(1) << 32) &&
                     (mode == kModeCr || mode == kModeClt);
    SectorDev sm = s;
    sm.mode = mode;
    return with_mode(mode, s.n_sites, [&](auto l, auto m) {
        using L = decltype(l);
        constexpr int MODE = decltype(m)::value;
        if constexpr (std::is_same_v<L, uint32_t> && (MODE == kModeCr || MODE == kModeClt))
            if (buf) return launch_hv_one<L, MODE, T, 1, true>(sm, B, h, st);
        return with_vb<T>(h.vb, [&](auto vb) { return launch_hv_one<L, MODE, T, decltype(vb)::value>(sm, B, h, st); });
    });
}

}  // namespace ftlm
