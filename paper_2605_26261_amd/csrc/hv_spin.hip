// General-spin kernels (local spin s = two_s / 2 > 1/2; Sec. 2, Eqs. 11-17):
// the matrix-free multi-vector H.x (plain and with the Lanczos epilogue),
// the sector tables (basis, compressed lookup table over the d^N labels) and
// the index kernels (rank, unrank, neighbour lists). The spin-1/2 sectors
// keep their own kernels (hv_impl.hpp, sector.hip).
#include "hv_impl.hpp"
#include "lanczos_small.hpp"
#include "spin.hpp"
#include "spinruns.hpp"

namespace ftlm {

namespace {

// LDS of the general-spin row kernels (hv_spin_lds_bytes): FP64 scratch,
// ladder factors fu[a] = sqrt(s(s+1) - m(m+1)) (m = a - s) in FP64 and FP32,
// the cumulative dimension table (CR) or the powers d^p (CLT), and (CR) the
// two [site][lane] slabs Y_{+1}, Y_{-1} of each wave.
struct SpinLds {
    double* red;
    double* fu_d;
    float* fu_f;
    uint32_t* table;
    uint32_t* yp;
    uint32_t* ym;
};

__device__ __forceinline__ void stage_spin_table(uint32_t* dst, const SectorDev& S, int mode) {
    if (mode == kModeCr) {
        const int count = S.n_sites * S.bw * (S.two_s + 1);
        for (int i = threadIdx.x; i < count; i += blockDim.x) dst[i] = *gptr(S.binom + i);
    } else if (threadIdx.x < unsigned(S.n_sites)) {
        uint32_t p = 1;
        for (unsigned k = 0; k < threadIdx.x; ++k) p *= uint32_t(S.two_s + 1);
        dst[threadIdx.x] = p;
    }
}

// Lays out and fills the LDS (visible after the caller's next barrier).
template <int MODE>
__device__ __forceinline__ SpinLds spin_lds_setup(unsigned char* smem, const SectorDev& S) {
    SpinLds l;
    l.red = reinterpret_cast<double*>(smem);
    l.fu_d = reinterpret_cast<double*>(smem + hv_red_bytes());
    l.fu_f = reinterpret_cast<float*>(smem + hv_red_bytes() + 64);
    l.table = reinterpret_cast<uint32_t*>(smem + hv_red_bytes() + 96);
    uint32_t* slabs = reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(l.table) +
                                                  hv_spin_table_lds_bytes(S));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    l.yp = slabs + size_t(wave) * 2 * S.n_sites * 64 + lane;
    l.ym = l.yp + S.n_sites * 64;
    if (threadIdx.x < 8) {
        const double s = 0.5 * S.two_s, m = double(threadIdx.x) - s;
        const double v = s * (s + 1.0) - m * (m + 1.0);
        const double f = (int(threadIdx.x) <= S.two_s && v > 0.0) ? sqrt(v) : 0.0;
        l.fu_d[threadIdx.x] = f;
        l.fu_f[threadIdx.x] = float(f);
    }
    stage_spin_table(l.table, S, MODE);
    return l;
}

// Accumulates one row: the diagonal sum_b J_b m_lo m_hi and, per valid ladder
// term, (J_b / 2) * f * x[partner] (Eqs. 12-14). Partner indices are clamped
// into [0, D) like the spin-1/2 visitor's.
template <typename T, int VB, int SB = 1>
struct SpinGather {
    // column col0 of row 0 of x as bytes and the row stride in bytes, as in
    // the spin-1/2 visitor: one multiply-add per partner address
    const unsigned char* __restrict__ xb;
    uint32_t ldb;
    uint32_t last;
    const BondTable& B;
    T (&acc)[VB];
    T& dsum;
    __device__ __forceinline__ void diag(int b, T mm) { dsum += T(2) * bond_coef<T>(B, b) * mm; }
    __device__ __forceinline__ const T* row(uint32_t i) const {
        return reinterpret_cast<const T*>(xb + uint64_t(i) * ldb);
    }
    __device__ __forceinline__ void flip(int b, int, uint32_t idx, T f) {
        const T c = bond_coef<T>(B, b) * f;
        T v[VB];
        idx = idx < last ? idx : last;
        load_row<T, VB>(row(idx), v);
#pragma unroll
        for (int i = 0; i < VB; ++i) acc[i] += c * v[i];
    }
    // CR: two slots, each with the ladder terms of SB bonds, in flight
    // (spin_cr_row_pairs) at every width (SB = spin_slot_bonds). Against one
    // flip at a time, icosahedron M = 0: s = 5/2, one column 12.9 -> 8.4 ms;
    // s = 3, 8 columns 186 -> 165 ms.
    // CLT: the terms of kGroup bonds per group (spin_clt_row_groups); group
    // sizes of 1 to 4 bonds timed at s = 5/2 (one column: 9.1, 8.0, 7.4 and
    // 7.6 ms; 8 columns, Lanczos step: 30.3, 27.8, 26.3 and 26.7 ms; at 2 and
    // 4 columns two bonds were best or within 3 %).
    static constexpr bool kPairs = true;
    static constexpr int kSlotBonds = SB;
    static constexpr int kGroup = (VB == 1 || VB == 8) ? 3 : 2;
    // The two slots of kSlotBonds bonds: rows of x and their weights (J_b / 2
    // times the ladder factors for an existing term, else 0); term k is bond
    // b0 + k / 2. A missing term loads row 0.
    static constexpr int kTerms = 2 * kSlotBonds;
    T slot_a[kTerms][VB], slot_b[kTerms][VB];
    T w_a[kTerms], w_b[kTerms];
    __device__ __forceinline__ void clear_slots() {
#pragma unroll
        for (int g = 0; g < kTerms; ++g) {
            w_a[g] = w_b[g] = T(0);
#pragma unroll
            for (int i = 0; i < VB; ++i) slot_a[g][i] = slot_b[g][i] = T(0);
        }
    }
    __device__ __forceinline__ void load_slot(T (&slot)[kTerms][VB], T (&w)[kTerms], int b0,
                                              const uint32_t (&idx)[kTerms], const bool (&on)[kTerms],
                                              const T (&f)[kTerms]) {
#pragma unroll
        for (int g = 0; g < kTerms; ++g) {
            const uint32_t c = idx[g] < last ? idx[g] : last;
            load_row<T, VB>(row(on[g] ? c : 0u), slot[g]);
            const T cb = bond_coef<T>(B, b0 + g / 2);
            w[g] = on[g] ? cb * f[g] : T(0);
        }
    }
    __device__ __forceinline__ void add_slot(const T (&slot)[kTerms][VB], const T (&w)[kTerms]) {
#pragma unroll
        for (int g = 0; g < kTerms; ++g) {
#pragma unroll
            for (int i = 0; i < VB; ++i) acc[i] += w[g] * slot[g][i];
        }
    }
    __device__ __forceinline__ void load_slot_a(int b0, const uint32_t (&idx)[kTerms], const bool (&on)[kTerms],
                                                const T (&f)[kTerms]) {
        load_slot(slot_a, w_a, b0, idx, on, f);
    }
    __device__ __forceinline__ void load_slot_b(int b0, const uint32_t (&idx)[kTerms], const bool (&on)[kTerms],
                                                const T (&f)[kTerms]) {
        load_slot(slot_b, w_b, b0, idx, on, f);
    }
    __device__ __forceinline__ void add_slot_a() { add_slot(slot_a, w_a); }
    __device__ __forceinline__ void add_slot_b() { add_slot(slot_b, w_b); }
    // kGroup bonds b0, b0 + 1, ...: term k is bond b0 + k / 2, e = +1 for
    // even k; rows of the existing terms are loaded together, the others
    // stay zero under weight zero.
    __device__ __forceinline__ void group(int b0, const uint32_t (&idx)[2 * kGroup], const bool (&on)[2 * kGroup],
                                          const T (&f)[2 * kGroup]) {
        T v[2 * kGroup][VB];
#pragma unroll
        for (int k = 0; k < 2 * kGroup; ++k) {
#pragma unroll
            for (int i = 0; i < VB; ++i) v[k][i] = T(0);
            if (on[k]) load_row<T, VB>(row(idx[k] < last ? idx[k] : last), v[k]);
        }
#pragma unroll
        for (int k = 0; k < 2 * kGroup; ++k) {
            const T c = on[k] ? bond_coef<T>(B, b0 + k / 2) * f[k] : T(0);
#pragma unroll
            for (int i = 0; i < VB; ++i) acc[i] += c * v[k][i];
        }
    }
};

template <typename T>
__device__ __forceinline__ const T* ladder_factors(const SpinLds& l) {
    if constexpr (sizeof(T) == 4) return reinterpret_cast<const T*>(l.fu_f);
    else return reinterpret_cast<const T*>(l.fu_d);
}

template <int MODE, typename T, typename V>
__device__ __forceinline__ void spin_row(uint32_t t, const SectorDev& S, const BondTable& B, const SpinLds& l,
                                         V& v) {
    const T* fu = ladder_factors<T>(l);
    if constexpr (MODE == kModeCr) {
        const CumDim D{l.table, S.bw, S.two_s + 1};
        if constexpr (V::kPairs) spin_cr_row_pairs<T>(t, S.n_up, S.two_s, B, D, fu, l.yp, l.ym, v);
        else spin_cr_row<T>(t, S.n_up, S.two_s, B, D, fu, l.yp, l.ym, v);
    } else {
        const double inv_d = 1.0 / double(S.two_s + 1);
        if constexpr (V::kGroup > 0) spin_clt_row_groups<T>(t, S.two_s, B, S.basis, S.clt, l.table, fu, inv_d, v);
        else spin_clt_row<T>(t, S.two_s, B, S.basis, S.clt, l.table, fu, inv_d, v);
    }
}

// Bonds per slot of the two-slot CR pipeline (icosahedron, s = 5/2, M = 0):
// two bonds took the 8-column Lanczos step from 25.7 to 23.8 ms but the plain
// H.x at one column from 8.46 to 8.64 ms and at 8 columns from 22.9 to 23.9.
constexpr int spin_slot_bonds(int vb, int epi) { return (vb == 8 && epi == kEpiLanczos) ? 2 : 1; }

// Rows [row0, row0 + nrows) of y = H x (columns [col0, col0 + VB) of [D][ld]
// blocks) over the tiles of block `bid` of a (sub-)grid of G blocks, with the
// Lanczos epilogue of hv_body (w = hv_a H u_k - hv_b u_{k-1} and the FP64
// <u_k, w> sums per wave in wsum).
template <int MODE, typename T, int VB, int EPI>
__device__ __forceinline__ void hv_spin_body(const SectorDev& S, const BondTable& B, const SpinLds& l,
                                             const T* __restrict__ x, T* __restrict__ y, uint64_t ld, uint32_t col0,
                                             uint32_t row0, uint32_t nrows, uint32_t bid, uint32_t G, int shift,
                                             const T* ab, bool first, double* wsum) {
    const int wave = threadIdx.x >> 6;
    const uint32_t ntiles = (nrows + kBlock - 1) / kBlock;
    for_each_tile(ntiles, bid, G, shift, [&](uint32_t tile) {
        const uint32_t r = tile * kBlock + threadIdx.x;
        const bool valid = r < nrows;
        T xt[VB], out[VB];
        if (valid) {
            const uint32_t t = row0 + r;
            T acc[VB];
#pragma unroll
            for (int c = 0; c < VB; ++c) acc[c] = T(0);
            T diag = T(0);
            SpinGather<T, VB, spin_slot_bonds(VB, EPI)> vis{reinterpret_cast<const unsigned char*>(x + col0),
                                                            uint32_t(ld * sizeof(T)), S.dim - 1, B, acc, diag};
            spin_row<MODE, T>(t, S, B, l, vis);
            load_row<T, VB>(x + uint64_t(t) * ld + col0, xt);
            if constexpr (EPI == kEpiPlain && MODE == kModeCr) {
                // as in hv_body: a row whose slots met an infinity or a NaN in
                // row 0 is walked once more, loading its own terms only
                if (!all_finite<T, VB>(acc)) {
#pragma unroll
                    for (int c = 0; c < VB; ++c) acc[c] = T(0);
                    diag = T(0);
                    spin_cr_row<T>(t, S.n_up, S.two_s, B, CumDim{l.table, S.bw, S.two_s + 1}, ladder_factors<T>(l),
                                   l.yp, l.ym, vis);
                }
            }
#pragma unroll
            for (int c = 0; c < VB; ++c) out[c] = diag * xt[c] + acc[c];
            T* yrow = y + uint64_t(r) * ld + col0;
            if constexpr (EPI == kEpiLanczos) {
                T z[VB];
                if (!first) {
                    load_row<T, VB>(yrow, z);
                } else {
#pragma unroll
                    for (int c = 0; c < VB; ++c) z[c] = T(0);
                }
#pragma unroll
                for (int c = 0; c < VB; ++c) out[c] = ab[c] * out[c] - ab[VB + c] * z[c];
            }
            store_row<T, VB>(yrow, out);
        }
        if constexpr (EPI == kEpiLanczos) {
            double p[VB];
#pragma unroll
            for (int c = 0; c < VB; ++c) p[c] = valid ? double(xt[c]) * double(out[c]) : 0.0;
            wave_fold_columns<VB>(p, wsum + wave * VB);
        }
    });
}

template <int MODE, typename T, int VB>
__global__ __launch_bounds__(kBlock) void hv_spin_kernel(SectorDev S, BondTable B, HvLaunch h) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ BondTable Bs;
    stage_bonds(Bs, &B);
    const SpinLds l = spin_lds_setup<MODE>(smem, S);
    __syncthreads();
    hv_spin_body<MODE, T, VB, kEpiPlain>(S, Bs, l, static_cast<const T*>(h.x), static_cast<T*>(h.y), h.ld, h.col0,
                                         h.row0, h.nrows, blockIdx.x, gridDim.x, h.super_shift, nullptr, false, nullptr);
}

// First half of a Lanczos step over the sectors of the launch, as
// hv_lanczos_kernel does it for spin 1/2: a persistent grid taking
// (sector, item) pairs from the per-XCD queue, partials in per-item slots,
// alpha summed by the last workgroup to leave.
template <int MODE, typename T, int VB>
__global__ __launch_bounds__(kBlock) void hv_spin_lanczos_kernel(LanczosLaunch a) {
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
        const SpinLds l = spin_lds_setup<MODE>(smem, S);
        double* wsum = l.red;
        for (int i = threadIdx.x; i < kWaves * VB; i += kBlock) wsum[i] = 0.0;
        __syncthreads();
        const T* x = uniform(block_of<T>(a, sw.u[(step - 1) & 1], S.dim));
        T* y = uniform(block_of<T>(a, sw.u[step & 1], S.dim));
        hv_spin_body<MODE, T, VB, kEpiLanczos>(S, B, l, x, y, a.block_ld, a.col0 - a.block0, 0, S.dim, local, uniform(sw.items),
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

// ---- by runs -----------------------------------------------------------------

template <typename T>
__device__ __forceinline__ HighDim stage_spin_runs(unsigned char* smem, const SectorDev& S, const SpinLow& L,
                                                   PairTable<T>& pairs) {
    // two ranks a word (after an odd count the table has two bytes of padding)
    uint32_t* rank = reinterpret_cast<uint32_t*>(smem);
    const uint32_t* src = reinterpret_cast<const uint32_t*>(L.rank);
    const int words = int(spin_low_strings(L.d) + 1) / 2;
    for (int i = threadIdx.x; i < words; i += blockDim.x) rank[i] = *gptr(src + i);
    uint32_t* dims = reinterpret_cast<uint32_t*>(smem + spin_runs_rank_bytes(S));
    const int per = S.bw * L.d, count = (S.n_sites - L.sites) * per;
    for (int i = threadIdx.x; i < count; i += blockDim.x) dims[i] = *gptr(S.binom + L.sites * per + i);
    pairs.stage(S.two_s);
    return HighDim{dims, S.bw, L.d, L.sites};
}

// The plain H.x by runs: every wave takes `chunk` consecutive rows at a time.
//
// What bounds it: s = 5/2, 144,840,476 rows, one FP32 vector 8.4 -> 4.3 ms. The
// row-by-row kernel issues 2300 VALU instructions per 64 rows, half of them for
// the walk down the digits; by runs about half of them are left and the partner
// lines that miss L2 take as long (two columns 8.7 -> 5.6 ms, one FP64 9.6 -> 6.0).
template <typename T, int VB>
__global__ __launch_bounds__(kBlock) void hv_spin_runs_kernel(SectorDev S, BondTable B, HvLaunch h) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ BondTable Bs;
    __shared__ __align__(16) PairTable<T> pairs;
    stage_bonds(Bs, &B);
    const SpinLow L = spin_low(S);
    const HighDim D = stage_spin_runs(smem, S, L, pairs);
    __syncthreads();
    const uint32_t wave = uniform(threadIdx.x >> 6);
    const uint32_t block_rows = kWaves * h.chunk;
    const uint32_t ntiles = uint32_t((uint64_t(h.nrows) + block_rows - 1) / block_rows);
    for_each_tile(ntiles, blockIdx.x, gridDim.x, h.super_shift, [&](uint32_t tile) {
        const uint64_t r0 = uint64_t(tile) * block_rows + uint64_t(wave) * h.chunk;
        if (r0 >= h.nrows) return;
        const uint32_t n = h.nrows - uint32_t(r0) < h.chunk ? h.nrows - uint32_t(r0) : h.chunk;
        const uint32_t pos = h.row0 + uint32_t(r0);
        spin_run_rows<T, VB, 2>(
            S, Bs, reinterpret_cast<const uint16_t*>(smem), D, L, pairs.v, static_cast<const T*>(h.x),
            static_cast<T*>(h.y), h.ld, h.col0, h.row0, pos, pos + n);
    });
}

// The Lanczos step's H.x of a small sector (small_lanczos).
template <int MODE, typename T, int VB, int NT>
__global__ __launch_bounds__(NT) void hv_spin_small_lanczos_kernel(LanczosLaunch a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ BondTable B;
    small_lanczos<T, VB, NT>(a, B, smem, [&](const SectorDev& S, uint32_t col0) {
        const SpinLds l = spin_lds_setup<MODE>(smem, S);
        return [=](uint32_t t, const T* x, T* y, const T* ab, bool first, double (&prod)[VB]) {
            T acc[VB], xt[VB], out[VB];
#pragma unroll
            for (int c = 0; c < VB; ++c) acc[c] = T(0);
            T diag = T(0);
            SpinGather<T, VB, spin_slot_bonds(VB, kEpiLanczos)> vis{
                reinterpret_cast<const unsigned char*>(x + col0), uint32_t(a.block_ld * sizeof(T)), S.dim - 1, B, acc, diag};
            spin_row<MODE, T>(t, S, B, l, vis);
            load_row<T, VB>(x + uint64_t(t) * a.block_ld + col0, xt);
#pragma unroll
            for (int c = 0; c < VB; ++c) out[c] = diag * xt[c] + acc[c];
            T* yrow = y + uint64_t(t) * a.block_ld + col0;
            lanczos_epilogue<T, VB>(xt, out, yrow, ab, first, prod);
            store_row<T, VB>(yrow, out);
        };
    });
}

template <typename F>
hipError_t with_spin_vb(int vb, F&& f) {
    switch (vb) {
        case 1: return f(std::integral_constant<int, 1>{});
        case 2: return f(std::integral_constant<int, 2>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 8: return f(std::integral_constant<int, 8>{});
        default: return hipErrorInvalidValue;
    }
}

template <typename K>
hipError_t allow_lds(K kern, size_t lds) {
    if (lds > 65536)
        return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   int(lds));
    return hipSuccess;
}

// ---- sector tables and index kernels -----------------------------------------

constexpr int kThreads = 256;

inline unsigned blocks_for(uint64_t n) {
    uint64_t b = (n + kThreads - 1) / kThreads;
    return unsigned(b > 1048576 ? 1048576 : (b == 0 ? 1 : b));
}

__device__ __forceinline__ uint64_t gid() { return uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; }
__device__ __forceinline__ uint64_t gstride() { return uint64_t(gridDim.x) * blockDim.x; }

__device__ __forceinline__ uint64_t digits_to_label(uint64_t dig, int n_sites, uint64_t d) {
    uint64_t n = 0;
    for (int p = n_sites - 1; p >= 0; --p) n = n * d + uint64_t(digit_of(dig, p));
    return n;
}

// basis[t] = the t-th sector label (one unrank per state).
__global__ __launch_bounds__(kThreads) void build_basis_spin_kernel(SectorDev S, uint32_t* basis) {
    extern __shared__ uint32_t tab[];
    stage_spin_table(tab, S, kModeCr);
    __syncthreads();
    const CumDim D{tab, S.bw, S.two_s + 1};
    for (uint64_t t = gid(); t < S.dim; t += gstride()) {
        const uint64_t dig = spin_unrank_digits(uint32_t(t), S.n_sites, S.n_up, S.two_s, D);
        basis[t] = uint32_t(digits_to_label(dig, S.n_sites, uint64_t(S.two_s + 1)));
    }
}

// One compressed-lookup-table block of 32 labels per thread (Eqs. 18-19):
// mask bit j is set when label 32b + j < d^N has the sector's digit sum; the
// prefix is the number of sector labels below 32b.
__global__ __launch_bounds__(kThreads) void build_clt_spin_kernel(SectorDev S, CltEntry* clt, uint64_t nblocks) {
    extern __shared__ uint32_t tab[];
    stage_spin_table(tab, S, kModeCr);
    __syncthreads();
    const CumDim D{tab, S.bw, S.two_s + 1};
    const uint32_t d = uint32_t(S.two_s + 1);
    for (uint64_t b = gid(); b < nblocks; b += gstride()) {
        uint32_t mask = 0;
        for (uint32_t j = 0; j < 32; ++j) {
            const uint64_t label = b * 32 + j;
            if (label >= S.n_labels) break;
            int sum = 0;
            (void)label_digits64(label, S.n_sites, d, &sum);
            if (sum == S.n_up) mask |= 1u << j;
        }
        int sum = 0;
        const uint64_t dig = label_digits64(b * 32, S.n_sites, d, &sum);
        clt[b].mask = mask;
        clt[b].prefix = spin_rank_digits(dig, S.n_sites, S.n_up, D);
    }
}

template <int MODE>
__global__ __launch_bounds__(kThreads) void rank_spin_kernel(SectorDev S, const uint64_t* labels, uint64_t* idx,
                                                             uint64_t n) {
    extern __shared__ uint32_t tab[];
    if (MODE == kModeCr) stage_spin_table(tab, S, kModeCr);
    __syncthreads();
    const CumDim D{tab, S.bw, S.two_s + 1};
    for (uint64_t i = gid(); i < n; i += gstride()) {
        const uint64_t x = labels[i];
        uint64_t out = ~uint64_t(0);
        if (x < S.n_labels) {
            if (MODE == kModeClt) {
                const uint32_t r = clt_lookup(S.clt, uint32_t(x));
                if (r != kNone32) out = r;
            } else {
                int sum = 0;
                const uint64_t dig = label_digits64(x, S.n_sites, uint32_t(S.two_s + 1), &sum);
                if (sum == S.n_up) out = spin_rank_digits(dig, S.n_sites, S.n_up, D);
            }
        }
        idx[i] = out;
    }
}

template <int MODE>
__global__ __launch_bounds__(kThreads) void unrank_spin_kernel(SectorDev S, const uint64_t* idx, uint64_t* labels,
                                                               uint64_t n) {
    extern __shared__ uint32_t tab[];
    if (MODE == kModeCr) stage_spin_table(tab, S, kModeCr);
    __syncthreads();
    const CumDim D{tab, S.bw, S.two_s + 1};
    for (uint64_t i = gid(); i < n; i += gstride()) {
        const uint64_t t = idx[i];
        uint64_t out = ~uint64_t(0);
        if (t < S.dim) {
            if (MODE == kModeClt) {
                out = S.basis[t];
            } else {
                const uint64_t dig = spin_unrank_digits(uint32_t(t), S.n_sites, S.n_up, S.two_s, D);
                out = digits_to_label(dig, S.n_sites, uint64_t(S.two_s + 1));
            }
        }
        labels[i] = out;
    }
}

// Partner indices of every (row, bond, ladder term) through the same row
// functions as the H.x: entry [row][2 b] is the source with a_i + 1, a_j - 1
// and [row][2 b + 1] the one with a_i - 1, a_j + 1, for the caller's bond b
// = (i, j), i < j; FTLM_NONE where the term does not exist.
struct SpinNeighbors {
    uint64_t* out;
    const BondTable& B;
    static constexpr bool kPairs = false;
    static constexpr int kGroup = 0;  // one term at a time
    __device__ __forceinline__ void diag(int, float) {}
    __device__ __forceinline__ void flip(int b, int e, uint32_t idx, float) { out[2 * B.orig(b) + e] = idx; }
};

template <int MODE>
__global__ __launch_bounds__(kBlock) void neighbors_spin_kernel(SectorDev S, BondTable B, uint64_t t0,
                                                                uint64_t count, uint64_t* out) {
    extern __shared__ __align__(16) unsigned char smem[];
    const SpinLds l = spin_lds_setup<MODE>(smem, S);
    __syncthreads();
    for (uint64_t r = gid(); r < count; r += gstride()) {
        uint64_t* row = out + r * uint64_t(2 * B.n_bonds);
        for (int k = 0; k < 2 * B.n_bonds; ++k) row[k] = ~uint64_t(0);
        SpinNeighbors v{row, B};
        spin_row<MODE, float>(uint32_t(t0 + r), S, B, l, v);
    }
}

}  // namespace

// Whether a product goes by runs: rows of up to 8 bytes (wider ones are bound by
// the lines they miss: s = 5/2, M = 0, four FP32 columns 10.4 ms row by row, 11.3
// by runs), from 2^23 of them (s = 3/2, 1.7 million: 104 against 111 us), at least
// 192 to a run on average. Icosahedron, FP32, one column: s = 2, M = 0 with 260 a
// run 1100 -> 838 us, M = 6 with 130 564 against 764; s = 5/2, M = 8 with 220 3484
// -> 2288, M = 12 with 85 1442 -> 1299 (with the compressed table 925). A share
// of the rows needs 2^31 / (rows to a run) of them: s = 2, M = 0, 2^16 rows 43
// against 16 us row by row, 2^22 265 against 242, 2^23 393 against 477; s = 5/2 with
// 517 a run 2^16 60 against 17, 2^22 221 against 251.
static bool spin_by_runs(const SectorDev& s, size_t row_bytes, uint32_t nrows) {
    const int d = s.two_s + 1, low = spin_low_sites(d), nh = s.n_sites - low;
    if (d > 6 || nh <= 0 || row_bytes > 8 || s.dim < (1u << 23)) return false;
    // high patterns that leave the low sites a digit sum they can have
    double count[kMaxSpinSites * kMaxTwoS + 1] = {1.0};
    for (int q = 0; q < nh; ++q) {
        double window = 0.0, old[kMaxTwoS + 1] = {};
        for (int k = 0; k <= (q + 1) * s.two_s; ++k) {
            const double c = k <= q * s.two_s ? count[k] : 0.0;
            window += c - old[k % d];
            old[k % d] = c;
            count[k] = window;
        }
    }
    double runs = 0.0;
    for (int k = 0; k <= nh * s.two_s && k <= s.n_up; ++k)
        if (s.n_up - k <= low * s.two_s) runs += count[k];
    if (nrows != s.dim && double(nrows) * double(s.dim) < 2147483648.0 * runs) return false;
    return double(s.dim) >= 192.0 * runs;
}

template <typename T, int VB>
hipError_t launch_hv_spin_runs(const SectorDev& s, const BondTable& B, HvLaunch h, hipStream_t st) {
    constexpr uint32_t kStep = 128, kChunk = 512;
    uint32_t steps = h.nrows / (8192u * kStep);
    steps = steps < 1 ? 1 : steps > kChunk / kStep ? kChunk / kStep : steps;
    h.chunk = steps * kStep;
    const uint64_t blocks = (uint64_t(h.nrows) + kWaves * h.chunk - 1) / (uint64_t(kWaves) * h.chunk);
    const uint64_t most = VB * sizeof(T) <= 4 ? 8192 : uint64_t(1) << 30;
    h.grid = int(blocks < 8 ? blocks : blocks < most ? (blocks + 7) & ~uint64_t(7) : most);
    h.super_shift = plain_super_shift(blocks, 6);
    const size_t lds = spin_runs_lds(s);
    auto kern = hv_spin_runs_kernel<T, VB>;
    hipError_t e = allow_lds(kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(unsigned(h.grid)), dim3(kBlock), lds, st, s, B, h);
    return hipGetLastError();
}

// Tiles from which on wide rows take one tile a block: 4096; ranked, with few terms,
// rows of up to 32 bytes 16384 (s = 5/2, M = 16, 13,889 tiles, 8 FP32 columns 384 us
// one tile a block, 331 on the persistent grid, but 418 and 517 with the table; s = 2,
// M = 6, 37,313 tiles 802 and 934). A new block stages its tables while the others on
// its CU work: with two, for the LDS they take, the persistent grid is the faster at
// every size (s = 7/2, 12 sites, 15 down steps, 28,689 tiles, 8 and 16 FP32 columns
// 709 and 2102 us, 1085 and 2708 one tile a block), with three for rows of up to 32
// bytes that are no part of wider ones, to 2^18 tiles (s = 3, 19 down steps, 151,135
// tiles 3.2 and 4.0 ms; s = 2, 433,423 tiles 13.3 and 11.7; 16 columns, two launches,
// s = 7/2, 63,147 tiles 6.3 and 5.0).
static uint32_t spin_few_tiles(const SectorDev& s, size_t row_bytes, bool whole, size_t lds) {
    const size_t used = (lds + sizeof(BondTable) + 1279) / 1280 * 1280;  // LDS goes out in 1280 bytes
    if (3 * used > 163840) return 1u << 30;
    if (row_bytes > 32 || !whole) return 4096;
    if (4 * used > 163840) return 1u << 18;
    return s.mode == kModeCr && few_flips(s.n_up, s.n_sites * s.two_s) ? 16384 : 4096;
}

hipError_t launch_hv_spin(const SectorDev& s, const BondTable& B, const HvLaunch& h0, hipStream_t st) {
    HvLaunch h = h0;
    const size_t row_bytes = size_t(h.vb) * (h.dtype == 0 ? 4 : 8);
    if (spin_by_runs(s, row_bytes, h.nrows)) {
        if (h.dtype != 0) return launch_hv_spin_runs<double, 1>(s, B, h, st);
        return h.vb == 1 ? launch_hv_spin_runs<float, 1>(s, B, h, st) : launch_hv_spin_runs<float, 2>(s, B, h, st);
    }
    const size_t lds = hv_spin_lds_bytes(s);
    walk_schedule(row_bytes, spin_few_tiles(s, row_bytes, h.ld == uint64_t(h.vb), lds), s.mode != kModeCr, h);
    auto go = [&](auto tt, auto mm) {
        using T = decltype(tt);
        constexpr int MODE = decltype(mm)::value;
        return with_spin_vb(h.vb, [&](auto vb) {
            auto kern = hv_spin_kernel<MODE, T, decltype(vb)::value>;
            hipError_t e = allow_lds(kern, lds);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(kern, dim3(unsigned(h.grid)), dim3(kBlock), lds, st, s, B, h);
            return hipGetLastError();
        });
    };
    const auto cr = std::integral_constant<int, kModeCr>{};
    const auto clt = std::integral_constant<int, kModeClt>{};
    if (h.dtype == 0) return s.mode == kModeCr ? go(float{}, cr) : go(float{}, clt);
    return s.mode == kModeCr ? go(double{}, cr) : go(double{}, clt);
}

hipError_t launch_hv_lanczos_spin(const LanczosLaunch& a, size_t lds, hipStream_t st) {
    if (!a.queue || a.items <= 0) return hipErrorInvalidValue;  // the queue counters are required
    const size_t small = small_lanczos_lds(a, lds, 2 * hv_slab_lds_bytes(a.n_sites, a.mode));
    if (by_small_lanczos(a, small)) {
        auto narrow = [&](auto tt, auto mm) {
            using T = decltype(tt);
            constexpr int MODE = decltype(mm)::value;
            return with_small_shape(a, [&](auto vb, auto nt) {
                constexpr int VB = decltype(vb)::value;
                return launch_small_lanczos(hv_spin_small_lanczos_kernel<MODE, T, VB, decltype(nt)::value>, VB, a, small,
                                            st);
            });
        };
        const auto cr = std::integral_constant<int, kModeCr>{};
        const auto clt = std::integral_constant<int, kModeClt>{};
        if (a.dtype == 0) return a.mode == kModeCr ? narrow(float{}, cr) : narrow(float{}, clt);
        return a.mode == kModeCr ? narrow(double{}, cr) : narrow(double{}, clt);
    }
    auto go = [&](auto tt, auto mm) {
        using T = decltype(tt);
        constexpr int MODE = decltype(mm)::value;
        return with_spin_vb(a.vb, [&](auto vb) {
            auto kern = hv_spin_lanczos_kernel<MODE, T, decltype(vb)::value>;
            const size_t bytes = lds < kGridSumLds ? kGridSumLds : lds;  // the final sums reuse the block's LDS
            hipError_t e = allow_lds(kern, bytes);
            if (e != hipSuccess) return e;
            int grid = 0;
            e = persistent_grid(reinterpret_cast<const void*>(kern), kBlock, bytes, a.items, &grid);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(kern, dim3(unsigned(grid)), dim3(kBlock), bytes, st, a);
            return hipGetLastError();
        });
    };
    const auto cr = std::integral_constant<int, kModeCr>{};
    const auto clt = std::integral_constant<int, kModeClt>{};
    if (a.dtype == 0) return a.mode == kModeCr ? go(float{}, cr) : go(float{}, clt);
    return a.mode == kModeCr ? go(double{}, cr) : go(double{}, clt);
}

static size_t spin_table_bytes(const SectorDev& s) {
    return size_t(s.n_sites) * size_t(s.bw) * size_t(s.two_s + 1) * 4;
}

hipError_t launch_build_basis_spin(const SectorDev& s, hipStream_t st) {
    hipLaunchKernelGGL(build_basis_spin_kernel, dim3(blocks_for(s.dim)), dim3(kThreads), spin_table_bytes(s), st, s,
                       const_cast<uint32_t*>(s.basis));
    return hipGetLastError();
}

hipError_t launch_build_clt_spin(const SectorDev& s, hipStream_t st) {
    const uint64_t nb = (s.n_labels + 31) / 32;
    hipLaunchKernelGGL(build_clt_spin_kernel, dim3(blocks_for(nb)), dim3(kThreads), spin_table_bytes(s), st, s,
                       const_cast<CltEntry*>(s.clt), nb);
    return hipGetLastError();
}

hipError_t launch_rank_spin(const SectorDev& s, const uint64_t* labels, uint64_t* idx, uint64_t n, hipStream_t st) {
    if (s.mode == kModeCr)
        hipLaunchKernelGGL(rank_spin_kernel<kModeCr>, dim3(blocks_for(n)), dim3(kThreads), spin_table_bytes(s), st, s,
                           labels, idx, n);
    else
        hipLaunchKernelGGL(rank_spin_kernel<kModeClt>, dim3(blocks_for(n)), dim3(kThreads), 0, st, s, labels, idx, n);
    return hipGetLastError();
}

hipError_t launch_unrank_spin(const SectorDev& s, const uint64_t* idx, uint64_t* labels, uint64_t n,
                              hipStream_t st) {
    if (s.mode == kModeCr)
        hipLaunchKernelGGL(unrank_spin_kernel<kModeCr>, dim3(blocks_for(n)), dim3(kThreads), spin_table_bytes(s), st,
                           s, idx, labels, n);
    else
        hipLaunchKernelGGL(unrank_spin_kernel<kModeClt>, dim3(blocks_for(n)), dim3(kThreads), 0, st, s, idx, labels,
                           n);
    return hipGetLastError();
}

hipError_t launch_neighbors_spin(const SectorDev& s, const BondTable& B, uint64_t t0, uint64_t count, uint64_t* out,
                                 hipStream_t st) {
    const size_t lds = hv_spin_lds_bytes(s);
    if (s.mode == kModeCr) {
        hipError_t e = allow_lds(neighbors_spin_kernel<kModeCr>, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(neighbors_spin_kernel<kModeCr>, dim3(blocks_for(count)), dim3(kBlock), lds, st, s, B, t0,
                           count, out);
    } else {
        hipError_t e = allow_lds(neighbors_spin_kernel<kModeClt>, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(neighbors_spin_kernel<kModeClt>, dim3(blocks_for(count)), dim3(kBlock), lds, st, s, B, t0,
                           count, out);
    }
    return hipGetLastError();
}

}  // namespace ftlm
