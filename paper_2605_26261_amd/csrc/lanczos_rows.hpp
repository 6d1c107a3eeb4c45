// First half of a Lanczos step over FP32 vectors (spin 1/2): the H.x with the
// Lanczos epilogue on consecutive work items, row by row or by runs.
#pragma once

#include "hv_impl.hpp"

namespace ftlm {

// Threads per workgroup of the kernels below: eight waves, or four
// - at 32 columns, whose registers leave room for eight waves per CU: two
//   workgroups take turns at their barriers (a step of 18 and 20 sites, half up, 55.0
//   and 133 us, 57.0 and 137 with eight waves; 16 columns were 6 % slower with four);
// - at 20 columns where less than a third of the spins are up, or down: twelve
//   waves per CU hide more of the few partner loads (22 sites, 6 up: 54.2 and 55.0
//   us; in a plan split that way, 30 sites, 9 up: 3.65 and 3.90 ms);
// - above 34 sites row by row, where the Y values of eight waves would leave a
//   CU one workgroup.
// The sums over a launch keep the order of eight waves.
inline int row_threads(int path, int n_sites, int n_up, int vb) {
    const int few = n_up < n_sites - n_up ? n_up : n_sites - n_up;
    return vb >= 32 || (vb == 20 && 3 * few < n_sites) || (n_sites > 34 && path == kModeCr) ? 256 : 512;
}

// How the rows are walked: an index map of the row-by-row visitor, or by runs.
constexpr int kPathRuns = 16;

// By runs: rows that a lane holds at a time (as in run_shape, except that one
// column takes two: with four 4.46 ms at N = 30, with two 3.90), and the slots
// of a work item, log2 (the other paths take one). What is found once for a run
// serves a wave's part of the item, an eighth; longer items loosen the front of
// rows in flight, which costs wide rows more than they gain. Icosidodecahedron,
// N = 30, slots of 1024 rows: one column 4.32 ms with one slot, 3.90, 3.58 and
// 3.37 with 2, 4 and 8; two columns 6.15, 5.75, 5.62 with 1, 2 and 4; four 8.87,
// 8.33, 8.51 with 1, 2 and 4; eight 16.7, 17.4, 18.8 with 1, 2 and 4. An
// item gets no longer than leaves 4096 of them (28 sites, 18 up, one column:
// 0.40 ms with 6400 items, 0.46 with 3200), but at least a lane's rows for
// every wave.
constexpr int run_lane_rows(int vb) { return vb <= 4 ? 2 : 1; }
constexpr int run_item_log(int vb) { return vb == 1 ? 3 : vb == 2 ? 2 : vb <= 4 ? 1 : 0; }
// 64-row groups of an item at most
constexpr int item_groups(int path, int vb) { return 16 << (path == kPathRuns ? run_item_log(vb) : 0); }

// LDS of the kernels: the binomial table (the widest of the launch's sectors), then
// a [site][lane] slab of Y values per wave (ranking); by runs the rank table and
// the binomial table. At least what the final sums need. (64 sites, 5 up: with room
// for any table, 17 KB, one workgroup a CU and 28.0 ms for eight columns, 16.2 with two.)
inline size_t lanczos_rows_lds(int path, int n_sites, int max_bw, int low_bits, int threads) {
    const size_t binom = (size_t(n_sites) * size_t(max_bw) * 4 + 15) & ~size_t(15);
    size_t n = 0;
    if (path == kPathRuns) n = (size_t(2) << low_bits) + binom;
    else if (path == kModeCr) n = binom + size_t(threads) * size_t(n_sites) * 4;
    return n < kGridSumLds ? kGridSumLds : n;
}

// One Lanczos step's H.x over every sector of the launch (one sector, all
// sectors of a plan, or a server round): w = H q_k - beta_{k-1} q_{k-1} and
// the FP64 partials of <u_k, w>, summed in slot order into alpha_k (and the
// update coefficient). A sector whose chains have all stopped is skipped.
//
// What bounds it. Wide blocks: the partner rows that miss L2 (that path gives 7
// TB/s), so items are consecutive rows and are handed out in their order, which
// keeps the rows in flight one compact front; strided items, each sweeping the
// whole sector, share fewer partners. N = 30: 8 columns 19.0 -> 16.7 ms, 16
// 41.4 -> 36.7, 20 56.8 -> 50.6 (plain H.x 14.3, 31.2, 38.9: its blocks end in
// order and leave at once). Narrow ones: the instructions that index the
// partners, which runs save (one column 7.9 -> 3.4 ms, two 8.1 -> 5.6, four 9.7
// -> 8.3). Small sectors: the length of one workgroup's work and the end of the
// launch (352,716 rows, 16 columns: 144 -> 83 us; 48,620 rows, 8 columns: 63 ->
// 21 us).
//
// The grid is persistent. Each workgroup starts with the item of its own
// number and then takes the next one from its XCD's counter, fetched while the
// current item runs; a sector's bonds, binomials and scalars are staged when it
// changes. A wave takes its eighth of the item, 64 rows at a time; the products
// of 64 rows are folded in the wave, and a slot's groups of 64 rows are added in
// order, so which workgroup ran an item, how long items are, the path and the
// launch width change no sum. The last workgroup to leave (queue_exit) sums
// every sector's slots. What all lanes share goes through uniform(): without it
// the compiler kept pointers and the sector in vector registers and the branches
// on them divergent (8 columns by runs: 133 registers, 103 with it).
template <typename L, int PATH, typename T, int VB, int NT>
__global__ __launch_bounds__(NT) void lanczos_rows_kernel(LanczosLaunch a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int flag;
    __shared__ uint32_t next[2];
    __shared__ BondTable B;
    __shared__ T ab[2 * VB];
    __shared__ double psum[item_groups(PATH, VB) * VB];
    constexpr int kRowWaves = NT / 64;
    constexpr bool kRuns = PATH == kPathRuns;
    constexpr int R = kRuns ? run_lane_rows(VB) : 1;
    const SecWork* secs = a.secs;
    const uint32_t xcd = blockIdx.x & 7u, grid8 = gridDim.x >> 3;
    const int lane = threadIdx.x & 63;
    const uint32_t wave = uniform(threadIdx.x >> 6);
    uint32_t* low = reinterpret_cast<uint32_t*>(smem);
    uint32_t* binom = low;
    if constexpr (kRuns) {
        const uint32_t* src = reinterpret_cast<const uint32_t*>(kLow.rank);
        for (int i = threadIdx.x; i < (1 << a.low_bits) / 2; i += NT) low[i] = *gptr(src + i);
        binom = low + (1 << a.low_bits) / 2;
    }
    uint32_t* ylds = binom + ((a.n_sites * a.max_bw + 3) & ~3) + wave * uint32_t(a.n_sites) * 64u + uint32_t(lane);
    SectorDev S{};
    const T* x = nullptr;
    T* y = nullptr;
    bool first = false;
    int cur = -1;
    uint32_t k = blockIdx.x >> 3;
    for (int par = 0;; par ^= 1) {
        uint32_t local = 0;
        const int s = uniform(block_item(secs, a.nsec, xcd, k, a.item_log, &local));
        if (s < 0) break;
        local = uniform(local);
        uint32_t after = ~0u;
        if (!a.one_round && threadIdx.x == 0) after = grid8 + atomicAdd(a.queue + xcd, 1u);
        const SecWork& sw = secs[s];
        if (uniform(sw.state[1]) != 0 && local << a.item_log < uniform(sw.items)) {
            if (s != cur) {
                cur = s;
                const int step = uniform(sw.state[0]);
                S = uniform(sw.S);
                x = uniform(block_of<T>(a, sw.u[(step - 1) & 1], S.dim));
                y = uniform(block_of<T>(a, sw.u[step & 1], S.dim));
                first = step == 1;
                stage_bonds(B, sw.bonds, NT);
                stage_epilogue<T, VB>(ab, sw.chains + a.col0);
                if constexpr (kRuns || PATH == kModeCr) stage_binomials(binom, S.binom, S.n_sites * S.bw);
                __syncthreads();
            }
            const Binom C{binom, S.bw};
            // a wave's part: consecutive groups of 64 rows, each summed on its own
            const uint32_t slot = slot_rows(S.dim) / 64u, groups = slot << a.item_log;
            const uint32_t part = groups / kRowWaves < uint32_t(R) ? uint32_t(R) : groups / kRowWaves;
            const uint64_t r0 = (uint64_t(local) * groups + wave * part) * 64u;
            double* sums = psum + wave * part * VB;
            if (wave * part < groups) {
                for (uint32_t i = lane; i < part * VB; i += 64u) sums[i] = 0.0;
            }
            if (wave * part < groups && r0 < S.dim) {
                const uint32_t t0 = uint32_t(r0);
                const uint32_t end = S.dim - t0 < part * 64u ? S.dim : t0 + part * 64u;
                if constexpr (kRuns) {
                    const unsigned char* xb = reinterpret_cast<const unsigned char*>(x);
                    Run<L> run;
                    RunBonds<T> rb;
                    run.base = run.size = 0;
#pragma unroll 1
                    for (uint32_t p0 = t0;; p0 += 64u * R) {
                        const uint32_t stop = end - p0 < 64u * R ? end : p0 + 64u * R;
                        double prod[R][VB];
                        uint32_t lo = p0;
                        for (uint32_t pos = p0; pos < stop;) {
                            lo = pos;
                            if (pos - run.base >= run.size) {
                                run.find(pos, S, C, a.low_bits, lane);
                                rb.load(run, B, 0, a.low_bits, lane, xb, VB * sizeof(T), S.dim - 1);
                            }
                            const uint32_t lim = stop - run.base < run.size ? stop : run.base + run.size;
                            run_block<L, T, VB, R, kRunGroup, kEpiLanczos>(S, B, smem, a.low_bits, run, rb, x, y, VB, 0,
                                                                           0, p0, pos, lim, ab, first, prod);
                            pos = lim;
                        }
                        // rows of several runs: the products of the earlier
                        // ones come from the rows that were just written
                        // (kept in registers, they would hold them through
                        // every bond loop)
                        if (lo != p0) {
#pragma unroll
                            for (int i = 0; i < R; ++i) {
                                const uint32_t t = p0 + uint32_t(64 * i + lane);
                                if (t >= p0 && t < lo) {
                                    T u[VB], w[VB];
                                    load_row<T, VB>(x + uint64_t(t) * VB, u);
                                    load_row<T, VB>(y + uint64_t(t) * VB, w);
#pragma unroll
                                    for (int c = 0; c < VB; ++c) prod[i][c] = double(u[c]) * double(w[c]);
                                }
                            }
                        }
#pragma unroll
                        for (int i = 0; i < R; ++i, sums += VB) wave_fold_columns<VB, false>(prod[i], sums);
                        if (stop == end) break;
                    }
                } else {
#pragma unroll 1
                    for (uint32_t p0 = t0;; p0 += 64u) {
                        const uint32_t stop = end - p0 < 64u ? end : p0 + 64u;
                        double prod[VB];
#pragma unroll
                        for (int c = 0; c < VB; ++c) prod[c] = 0.0;
                        if (p0 + uint32_t(lane) < stop)
                            walk_row<L, PATH, T, VB>(p0 + uint32_t(lane), S, B, C, ylds, x, y, VB, 0, ab, first,
                                                     prod);
                        wave_fold_columns<VB, false>(prod, sums);
                        sums += VB;
                        if (stop == end) break;
                    }
                }
            }
            __syncthreads();
            const uint32_t j = threadIdx.x / VB, at = (local << a.item_log) + j;
            if (j < 1u << a.item_log && at < uniform(sw.items)) {
                const double* g = psum + j * slot * VB + threadIdx.x % VB;
                double t = 0.0;
                for (uint32_t i = 0; i < slot; ++i) t += g[i * VB];
                publish(sw.partials + size_t(at) * a.ld + a.col0 + threadIdx.x % VB, t);
            }
        }
        if (threadIdx.x == 0) next[par] = after;
        __syncthreads();
        k = uniform(next[par]);
    }
    if (queue_exit(a.queue, gridDim.x, &flag)) {
        double* red = reinterpret_cast<double*>(smem);
        for (int s = 0; s < a.nsec; ++s)
            if (uniform(secs[s].state[1]) != 0) finish_alpha<VB, NT, 512>(secs[s], a, secs[s].items, red);
    }
}

template <typename L, int PATH, typename T, int VB, int NT = 512>
hipError_t launch_lanczos_rows(LanczosLaunch a, hipStream_t st) {
    auto kern = lanczos_rows_kernel<L, PATH, T, VB, NT>;
    size_t lds = lanczos_rows_lds(PATH, a.n_sites, a.max_bw, a.low_bits, NT);
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
        if (e != hipSuccess) return e;
    }
    if (!a.queue || a.items <= 0) return hipErrorInvalidValue;  // the queue counters are required
    int resident = 0;
    hipError_t e = persistent_grid(reinterpret_cast<const void*>(kern), NT, lds, 1 << 20, &resident);
    if (e != hipSuccess) return e;
    // Two slots to an item where that saves a second, partly filled round
    // (22-site cluster, one column: 48 us with one slot, 37 with two).
    if (a.item_log == 0 && 2 * slot_rows(uint32_t(a.max_dim)) <= 64 * item_groups(PATH, VB) &&
        a.xcd_items * 8 > resident && a.xcd_pairs * 8 <= resident) {
        a.item_log = 1;
        a.xcd_items = a.xcd_pairs;
    }
    const int grid = std::min(resident, a.xcd_items * 8);
    a.one_round = grid == a.xcd_items * 8 ? 1 : 0;
    hipLaunchKernelGGL(kern, dim3(unsigned(grid)), dim3(NT), lds, st, a);
    return hipGetLastError();
}

// The path of a launch: by runs where a product of the sector would go that
// way (one sector; a plan's sectors reach from one row to millions, and its
// short-run sectors would end last), else row by row with the index map that a
// product would use.
inline int lanczos_path(LanczosLaunch& a) {
    SectorDev s{};
    s.n_sites = a.n_sites;
    s.n_up = a.n_up;
    s.mode = a.mode;
    s.dim = uint32_t(a.max_dim);
    const size_t row_bytes = size_t(a.vb) * sizeof(float);
    a.low_bits = run_shape(row_bytes).low_bits;
    a.item_log = 0;
    if (a.nsec == 1 && by_runs(s, row_bytes, 4.0, false, 6.0, 2.0)) {
        const uint32_t slots = sector_items(s.dim, true);
        a.item_log = run_item_log(a.vb);
        const uint32_t least = 512u * uint32_t(run_lane_rows(a.vb));
        while (a.item_log > 0 && (slots >> a.item_log) < 4096u && (slot_rows(s.dim) << (a.item_log - 1)) >= least)
            --a.item_log;
        a.xcd_items = int(xcd_items((slots + (1u << a.item_log) - 1u) >> a.item_log, 0));
        return kPathRuns;
    }
    const int mode = product_map(s, row_bytes, false, s.dim);
    return a.vb > 8 ? kModeCr : mode;
}

inline hipError_t launch_lanczos_rows_any(LanczosLaunch a, hipStream_t st) {
    const int path = lanczos_path(a);
    return with_vb<float>(a.vb, [&](auto vb) {
        constexpr int VB = decltype(vb)::value;
        const bool wide = a.n_sites > 32;
        if constexpr (VB <= 8) {
            if (path == kPathRuns)
                return wide ? launch_lanczos_rows<uint64_t, kPathRuns, float, VB>(a, st)
                            : launch_lanczos_rows<uint32_t, kPathRuns, float, VB>(a, st);
            if (path == kModeClt) return launch_lanczos_rows<uint32_t, kModeClt, float, VB>(a, st);
            if (path == kModeFull) return launch_lanczos_rows<uint32_t, kModeFull, float, VB>(a, st);
            if (path == kModeLin) return launch_lanczos_rows<uint32_t, kModeLin, float, VB>(a, st);
        }
        const bool four = row_threads(path, a.n_sites, a.n_up, VB) == 256;
        if (wide) {
            if (four) return launch_lanczos_rows<uint64_t, kModeCr, float, VB, 256>(a, st);
            if constexpr (VB < 32) return launch_lanczos_rows<uint64_t, kModeCr, float, VB>(a, st);
        }
        if constexpr (VB >= 20) {
            if (four) return launch_lanczos_rows<uint32_t, kModeCr, float, VB, 256>(a, st);
        }
        if constexpr (VB < 32) return launch_lanczos_rows<uint32_t, kModeCr, float, VB>(a, st);
        return hipErrorInvalidValue;  // not reached: 32 columns take four waves
    });
}

}  // namespace ftlm
