// Lanczos kernels over a list of sectors: start vectors and the second half
// of a Lanczos step (paper Sec. 2, the recursion after Eq. 3, without
// reorthogonalization). The first half of a step (w = H q_k - beta_{k-1}
// q_{k-1} and alpha_k) is lanczos_rows_kernel (FP32, spin 1/2), hv_lanczos_kernel
// or hv_spin_lanczos_kernel, for small sectors a kernel of lanczos_small.hpp;
// tiny_chain_kernel takes both halves of all steps. A launch covers one sector or
// every sector of a plan; each sector owns a contiguous range of blocks.
#include <math.h>

#include <algorithm>
#include <map>
#include <mutex>

#include "hv_impl.hpp"

namespace ftlm {

hipError_t persistent_grid(const void* kern, int threads, size_t lds, int items, int* grid) {
    static std::mutex mu;
    static std::map<std::pair<const void*, size_t>, int> cache;  // per kernel and LDS size
    int per_cu = 0;
    {
        std::lock_guard<std::mutex> lk(mu);
        auto it = cache.find({kern, lds});
        if (it != cache.end()) {
            per_cu = it->second;
        } else {
            hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, threads, lds);
            if (e != hipSuccess) return e;
            cache[{kern, lds}] = per_cu;
        }
    }
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    const int resident = ((std::max(1, per_cu) * cus + 7) / 8) * 8;
    const int cap = ((items + 7) / 8) * 8;
    *grid = std::max(8, std::min(resident, cap));
    return hipSuccess;
}

hipError_t launch_hv_lanczos(const LanczosLaunch& a, size_t lds, hipStream_t st) {
    if (a.two_s > 1) return launch_hv_lanczos_spin(a, lds, st);
    return a.dtype == 0 ? launch_lanczos_f32(a, st) : launch_lanczos_f64(a, lds, st);
}

namespace {

constexpr int kTinyThreads = 1024;
constexpr int kTinyTiles = 7;  // fewer than eight: one tile to a work item and to an update block
constexpr size_t kTinyLds = 152 * 1024;

constexpr uint64_t kGamma = 0x9e3779b97f4a7c15ull;

// SplitMix64's output function (Steele, Lea, Flood 2014).
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// Entry i of a start vector from the stream with key `key`: output i of the
// generator is mix64(key + (i + 1) * gamma).
__device__ __forceinline__ double start_entry(int dist, uint64_t key, uint64_t i, uint64_t sample) {
    if (dist == 0) {
        return (mix64(key + (i + 1) * kGamma) >> 63) ? -1.0 : 1.0;
    } else if (dist == 1) {
        const uint64_t u1 = mix64(key + (2 * i + 1) * kGamma);
        const uint64_t u2 = mix64(key + (2 * i + 2) * kGamma);
        const double a = double((u1 >> 11) + 1) * 0x1.0p-53;  // (0, 1]
        const double b = double(u2 >> 11) * 0x1.0p-53;        // [0, 1)
        return sqrt(-2.0 * log(a)) * cos(2.0 * 3.141592653589793 * b);
    }
    return i == sample ? 1.0 : 0.0;
}

// Writes columns [col0, col0 + vb) (vb <= CB) of every sector's start block
// u_1 and their FP64 norms; the last block of a sector turns the norms into
// each chain's initial scale s_1 = 1 / |u_1|. Bound by the arithmetic of an entry
// (FP64 log and cos of a Gaussian: 8 columns at N = 30 10.6 ms, 12.3 with a store
// per entry and the key read again for each), or by the launches: up to eight
// columns go together and a row is stored with wide accesses (9.7 million rows of
// 32 signs: 1.27 -> 0.51 ms). One column to four waves was slower (17.8 ms, 4-byte
// stores of four waves to each line).
template <typename T, int CB>
__global__ __launch_bounds__(kBlock) void start_kernel(LanczosLaunch a) {
    __shared__ double red[grid_sum_lds<CB>() / sizeof(double)];
    __shared__ int flag;
    uint32_t local = 0;
    const int s = sector_of_block(a.secs, a.nsec, blockIdx.x, &local);
    if (s < 0) return;
    const SecWork& sw = a.secs[s];
    const uint32_t dim = sw.S.dim;
    T* q = block_of<T>(a, sw.u[0], dim);
    const int nc = a.vb < CB ? a.vb : CB;
    double part[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) part[c] = 0.0;
    uint64_t key[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) key[c] = c < nc ? sw.keys[a.col0 + c] : 0;
    const uint32_t ntiles = (dim + kBlock - 1) / kBlock;
    for_each_tile(ntiles, local, sw.G, kXcdSuperShift, [&](uint32_t tile) {
        const uint32_t t = tile * kBlock + threadIdx.x;
        if (t >= dim) return;
        T* row = q + uint64_t(t) * a.block_ld + (a.col0 - a.block0);
        T v[CB];
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            v[c] = T(0);
            if (c < nc) {
                v[c] = T(start_entry(a.dist, key[c], t, sw.r0 + a.col0 + c));
                part[c] += double(v[c]) * double(v[c]);
            }
        }
        if (nc == CB) {
            store_row<T, CB>(row, v);
        } else {
#pragma unroll
            for (int c = 0; c < CB; ++c)
                if (c < nc) row[c] = v[c];
        }
    });
    block_sum<CB>(part, red, sw.partials + size_t(local) * a.ld + a.col0, nc);
    if (last_block(sw.ticket, sw.G, &flag)) {
        __shared__ double tot[grid_sum_slots<CB>()];
        grid_sum_cols<CB>(sw.partials, int(sw.G), int(a.ld), int(a.col0), nc, red, tot);
        if (threadIdx.x < 64) {  // one lane per column
            const bool mine = int(threadIdx.x) < nc;
            const double nrm = mine ? sqrt(tot[threadIdx.x]) : 0.0;
            if (mine) {
                Chain* ch = &sw.chains[a.col0 + threadIdx.x];
                ch->norm = nrm;
                ch->s_cur = nrm > 0.0 ? 1.0 / nrm : 0.0;
                ch->s_prev = 0.0;
                ch->beta_prev = 0.0;
                ch->amax = 0.0;
                ch->alpha = 0.0;
                ch->active = nrm > 0.0 ? 1 : 0;
                ch->steps = 0;
                chain_set_hv(ch);
            }
            const int started = __popcll(__ballot(nrm > 0.0));
            if (threadIdx.x == 0) {
                sw.state[1] += started;
                *sw.ticket = 0u;
            }
        }
    }
}

// beta_k = |w| of the chain in column col from |w|^2: records step k's
// coefficients, applies the stopping rule and sets the next step's scalars.
// Returns whether the chain stopped.
__device__ __forceinline__ bool finish_beta(Chain* ch, const SecWork& sw, int col, int step, double norm2, double eps) {
    if (!ch->active) return false;
    const double bk = sqrt(norm2);
    const double ak = ch->alpha;
    sw.alpha[size_t(col) * kMaxSteps + (step - 1)] = ak;
    sw.beta[size_t(col) * kMaxSteps + (step - 1)] = bk;
    const double amax = fmax(ch->amax, fmax(fabs(ak), ch->beta_prev));
    ch->amax = amax;
    ch->steps = step;
    // a non-finite coefficient ends the chain and marks it (the host reports
    // FTLM_E_NUMERIC); the comparison below is false for NaN, so without this
    // the chain would run on
    const bool fault = !(isfinite(ak) && isfinite(bk));
    if (fault) ch->fault = 1;
    const bool stopped = fault || step >= sw.m_eff || bk <= eps * amax;
    if (stopped) {
        ch->active = 0;
        ch->s_cur = 0.0;
        ch->s_prev = 0.0;
        ch->beta_prev = 0.0;
    } else {
        ch->s_prev = ch->s_cur;
        ch->s_cur = 1.0 / bk;
        ch->beta_prev = bk;
    }
    chain_set_hv(ch);
    return stopped;
}

// Second half of Lanczos step k for columns [col0, col0 + VB) of every
// sector:  w -= alpha_k q_k (q_k = s_k u_k),  beta_k = |w|,  u_{k+1} = w,
// with |w|^2 accumulated in FP64 per block and summed in fixed order by the
// sector's last block, which then records alpha_k and beta_k and applies the
// stopping rule: a chain stops after step k when k reaches min(M, D) or
// beta_k <= eps * max_{j<=k}(|alpha_j|, beta_{j-1}). A stopped chain gets
// zero scales, so its columns stay zero in every later step.
// Rows of 32 to 128 bytes (a multiple of 8) go through LDS: a tile's rows of u
// and w are contiguous, so they move with fully
// coalesced 16-byte accesses (8-byte ones for rows that are not a multiple of
// 16 bytes), while each thread still updates its own row (the same arithmetic
// and summation order as without the staging). With one thread per row, a
// vector access of rows that wide spans several cache lines per wave;
// narrower rows are already well coalesced. Rows of up to 96 bytes are staged
// a whole tile at a time, 128-byte rows half a tile at a time (two 256-row
// tiles would not fit the static LDS). A block loads its next chunk into
// registers before it stores the current one, so its reads stay in flight
// while it writes; every byte is touched once per step, so the accesses are
// non-temporal. Without the staging, 128-byte rows ran at under 1 TB/s and
// 40-byte rows at 4.0 TB/s; staged without the prefetch, 48-byte rows ran at
// 4.7 TB/s, and with it at 5.1 TB/s.
template <typename T, int VB>
__host__ __device__ constexpr bool update_staged() {
    return (VB * sizeof(T)) % 8 == 0 && VB * sizeof(T) >= 32 && VB * sizeof(T) <= 128;
}

template <typename T, int VB>
__host__ __device__ constexpr int update_stage_rows() {
    return VB * sizeof(T) <= 96 ? kBlock : kBlock / 2;
}

template <typename T, int VB>
__global__ __launch_bounds__(kBlock) void update_kernel(LanczosLaunch a) {
    __shared__ int flag;
    constexpr bool kStage = update_staged<T, VB>();
    constexpr int kStageRows = update_stage_rows<T, VB>();
    __shared__ __align__(16) T stage_u[kStage ? kStageRows * VB : 1];
    __shared__ __align__(16) T stage_w[kStage ? kStageRows * VB : 1];
    // the reductions come after the rows and reuse their LDS
    constexpr bool kOwnRed = sizeof(stage_w) < grid_sum_lds<VB>();
    __shared__ double own_red[kOwnRed ? grid_sum_lds<VB>() / sizeof(double) : 1];
    double* red = kOwnRed ? own_red : reinterpret_cast<double*>(stage_w);
    uint32_t local = 0;
    const int s = sector_of_block(a.secs, a.nsec, blockIdx.x, &local);
    if (s < 0) return;
    const SecWork& sw = a.secs[s];
    if (sw.state[1] == 0) return;
    const int step = sw.state[0];
    const uint32_t dim = sw.S.dim;
    const T* __restrict__ u = block_of<T>(a, sw.u[(step - 1) & 1], dim);
    T* __restrict__ w = block_of<T>(a, sw.u[step & 1], dim);
    // the update coefficients, read once (through a generic pointer the
    // compiler would re-read them after every store of the tile loop)
    T coef[VB];
#pragma unroll
    for (int c = 0; c < VB; ++c) {
        const Chain* ch = sw.chains + a.col0 + c;
        coef[c] = sizeof(T) == 4 ? T(ch->up_f) : T(ch->up_d);
    }
    double part[VB];
#pragma unroll
    for (int c = 0; c < VB; ++c) part[c] = 0.0;
    const uint32_t ntiles = (dim + kBlock - 1) / kBlock;
    if constexpr (kStage) {
        // copy unit: 16 bytes, or 8 for rows of an odd number of 8-byte words
        constexpr int kUnit = (VB * sizeof(T)) % 16 == 0 ? 4 : 2;
        using VU = uint32_t __attribute__((ext_vector_type(kUnit)));
        constexpr uint32_t kRowUnits = uint32_t(VB * sizeof(T)) / uint32_t(4 * kUnit);
        constexpr int kPer = int((uint32_t(kStageRows) * kRowUnits + kBlock - 1) / kBlock);
        VU* lu = reinterpret_cast<VU*>(stage_u);
        VU* lw = reinterpret_cast<VU*>(stage_w);
        // A chunk is rows [h0, h0 + hr) of one tile; the block walks its
        // tiles in tile_span's order. The next chunk's rows are loaded
        // into registers while the current chunk is stored.
        VU pu[kPer], pw[kPer];
        auto tile_rows = [&](uint32_t tile) {
            return dim - tile * kBlock < uint32_t(kBlock) ? dim - tile * kBlock : uint32_t(kBlock);
        };
        auto chunk_units = [&](uint32_t tile, uint32_t h0) {
            const uint32_t left = tile_rows(tile) - h0;
            return (left < uint32_t(kStageRows) ? left : uint32_t(kStageRows)) * kRowUnits;
        };
        auto fetch = [&](uint32_t tile, uint32_t h0) {
            const uint32_t n = chunk_units(tile, h0);
            const uint64_t r0 = uint64_t(tile) * kBlock + h0;
            const VU FTLM_GLOBAL* gu = gptr(reinterpret_cast<const VU*>(u + r0 * VB));
            const VU FTLM_GLOBAL* gw = gptr(reinterpret_cast<const VU*>(w + r0 * VB));
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const uint32_t i = threadIdx.x + uint32_t(k) * kBlock;
                if (i < n) {
                    pu[k] = __builtin_nontemporal_load(gu + i);
                    pw[k] = __builtin_nontemporal_load(gw + i);
                }
            }
        };
        const TileSpan sp = tile_span(ntiles, local, sw.G);
        uint32_t tile = sp.first, h0 = 0;
        if (tile < sp.end) fetch(tile, h0);
        while (tile < sp.end) {
            const uint32_t n = chunk_units(tile, h0);
            const uint32_t hr = n / kRowUnits;
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const uint32_t i = threadIdx.x + uint32_t(k) * kBlock;
                if (i < n) {
                    lu[i] = pu[k];
                    lw[i] = pw[k];
                }
            }
            __syncthreads();
            // each thread updates the row it owns (row threadIdx.x of the tile)
            if (threadIdx.x >= h0 && threadIdx.x < h0 + hr) {
                T* wr = stage_w + (threadIdx.x - h0) * VB;
                const T* ur = stage_u + (threadIdx.x - h0) * VB;
#pragma unroll
                for (int c = 0; c < VB; ++c) {
                    const T v = wr[c] - coef[c] * ur[c];
                    part[c] += double(v) * double(v);
                    wr[c] = v;
                }
            }
            __syncthreads();
            VU FTLM_GLOBAL* gw = gptr(reinterpret_cast<VU*>(w + (uint64_t(tile) * kBlock + h0) * VB));
            h0 += uint32_t(kStageRows);
            if (h0 >= tile_rows(tile)) {
                h0 = 0;
                tile += sp.step;
            }
            if (tile < sp.end) fetch(tile, h0);
            for (uint32_t i = threadIdx.x; i < n; i += kBlock) __builtin_nontemporal_store(lw[i], gw + i);
            __syncthreads();
        }
    } else {
        for_each_span_tile(ntiles, local, sw.G, [&](uint32_t tile) {
            const uint32_t t = tile * kBlock + threadIdx.x;
            if (t >= dim) return;
            T uu[VB], ww[VB];
            load_row<T, VB>(u + uint64_t(t) * VB, uu);
            T* wrow = w + uint64_t(t) * VB;
            load_row<T, VB>(wrow, ww);
#pragma unroll
            for (int c = 0; c < VB; ++c) {
                ww[c] = ww[c] - coef[c] * uu[c];
                part[c] += double(ww[c]) * double(ww[c]);
            }
            store_row<T, VB>(wrow, ww);
        });
    }
    __syncthreads();
    block_sum<VB>(part, red, sw.partials + size_t(local) * a.ld + a.col0, VB);
    if (last_block(sw.ticket, sw.G, &flag)) {
        __shared__ double tot[grid_sum_slots<VB>()];
        grid_sum_cols<VB>(sw.partials, int(sw.G), int(a.ld), int(a.col0), VB, red, tot);
        if (threadIdx.x < 64) {  // one lane per column
            bool stopped = false;
            if (threadIdx.x < VB) {
                const int col = int(a.col0 + threadIdx.x);
                stopped = finish_beta(&sw.chains[col], sw, col, step, tot[threadIdx.x], a.eps);
            }
            const int n = __popcll(__ballot(stopped));
            if (threadIdx.x == 0) {
                if (n) sw.state[1] -= n;
                if (a.last_chunk) sw.state[0] = step + 1;
                *sw.ticket = 0u;
            }
        }
    }
}

// Row gathers from a vector in LDS, one column (GatherVisitor's flip).
template <typename T>
struct LdsGather {
    const T* x;
    uint32_t last;
    const BondTable& B;
    T& acc;
    T& anti;
    __device__ __forceinline__ void flip(int b, uint32_t i) {
        const T c = bond_coef<T>(B, b);
        acc += c * x[i < last ? i : last];
        anti += c;
    }
    __device__ __forceinline__ void par(int) {}
};

// A row's partners, bond by bond (kNoPartner: the bond does not flip).
constexpr uint32_t kNoPartner = 0xffffu;
struct LdsPartners {
    uint16_t* p;  // of bond 0
    uint32_t stride, last;
    __device__ __forceinline__ void flip(int b, uint32_t i) { p[uint32_t(b) * stride] = uint16_t(i < last ? i : last); }
    __device__ __forceinline__ void par(int b) { p[uint32_t(b) * stride] = uint16_t(kNoPartner); }
};

// LDS of tiny_chain_kernel: both vectors, the binomial table, the Y values of
// its waves, and the rows' partners where they fit.
inline size_t tiny_chain_lds(uint64_t dim, int n_sites, size_t es) {
    return 2 * ((size_t(dim) * es + 15) & ~size_t(15)) + ((size_t(n_sites) * size_t(n_sites + 3) * 4 + 15) & ~size_t(15)) +
           size_t(kTinyThreads) * size_t(n_sites) * 4;
}
inline size_t tiny_partner_lds(uint64_t dim, int n_bonds) {
    return size_t(n_bonds) * size_t((dim + 63) & ~uint64_t(63)) * 2;
}

// Every step of one chain (blockIdx.x) of one sector (blockIdx.y) of at most
// kTinyTiles row tiles by one workgroup, both vectors in LDS from start to end.
//
// What bounds it: the latency of a row's gathers and of four barriers a step.
// Step by step 924 rows (24 bonds, 8 FP64 columns) took 21 us for two launches,
// each with its ticket and the gap after it; here a step takes 7.1 us with every
// row walked in every step and 4.2 with the partners, the same in all steps,
// found once (`partners`: they fit beside the rest).
//
// Up to seven row tiles each is a work item and a block of its own, so the sums
// are those of the step-by-step kernels: a wave's 64 rows by fold, a tile's four
// waves in order, the tiles by the fold of the first wave.
template <typename L, typename T>
__global__ __launch_bounds__(kTinyThreads) void tiny_chain_kernel(LanczosLaunch a, ChainBlocks blocks, int partners) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ BondTable B;
    __shared__ double psum[4 * kTinyTiles];
    __shared__ Chain chain;
    __shared__ double tot;
    const SecWork& sw = a.secs[blockIdx.y];
    const int col = int(blockIdx.x);
    a.block0 = blocks.first[col];
    a.block_ld = blocks.width[col];
    const SectorDev S = uniform(sw.S);
    const uint32_t dim = S.dim, groups = 4u * ((dim + kBlock - 1) / kBlock);
    const int lane = threadIdx.x & 63;
    const uint32_t wave = uniform(threadIdx.x >> 6);
    T* u0 = reinterpret_cast<T*>(smem);
    T* u1 = reinterpret_cast<T*>(smem + ((size_t(dim) * sizeof(T) + 15) & ~size_t(15)));
    uint32_t* binom = reinterpret_cast<uint32_t*>(smem + 2 * ((size_t(dim) * sizeof(T) + 15) & ~size_t(15)));
    uint32_t* ylds = binom + ((S.n_sites * S.bw + 3) & ~3) + wave * uint32_t(S.n_sites) * 64u + uint32_t(lane);
    stage_bonds(B, sw.bonds, kTinyThreads);
    stage_binomials(binom, S.binom, S.n_sites * S.bw);
    const T* src = block_of<T>(a, sw.u[0], dim) + (uint32_t(col) - a.block0);
    for (uint32_t t = threadIdx.x; t < dim; t += kTinyThreads) u0[t] = *gptr(src + uint64_t(t) * a.block_ld);
    if (threadIdx.x == 0) chain = sw.chains[col];
    __syncthreads();
    const Binom C{binom, S.bw};
    const T jsum4 = sizeof(T) == 4 ? T(B.jsum4_f) : T(B.jsum4_d);
    const uint32_t stride = (dim + 63u) & ~63u;
    const int n_bonds = uniform(B.n_bonds);
    uint16_t* const rows = reinterpret_cast<uint16_t*>(binom + ((S.n_sites * S.bw + 3) & ~3) + kTinyThreads * S.n_sites);
    if (partners) {
        for (uint32_t t = wave * 64u + uint32_t(lane); t < dim; t += kTinyThreads) {
            LdsPartners vis{rows + t, stride, dim - 1};
            cr_bonds<L, false>(t, L(0), S.n_up, B, C, ylds, vis);
        }
    }
    // the sums of the tiles' rows from those of their waves, by the first wave
    auto total = [&] {
        double t[1] = {0.0};
        if (uint32_t(lane) * 4u < groups)
            for (int w = 0; w < 4; ++w) t[0] += psum[4 * lane + w];
        wave_fold_columns<1, false>(t, &tot);
        __builtin_amdgcn_wave_barrier();
    };
#pragma unroll 1
    for (int step = 1; chain.active; ++step) {
        const T* x = (step & 1) ? u0 : u1;
        T* y = (step & 1) ? u1 : u0;
        const T ab[2] = {sizeof(T) == 4 ? T(chain.hv_a_f) : T(chain.hv_a_d),
                         sizeof(T) == 4 ? T(chain.hv_b_f) : T(chain.hv_b_d)};
        for (uint32_t g = wave; g < groups; g += kTinyThreads / 64) {
            const uint32_t t = g * 64u + uint32_t(lane);
            double prod[1] = {0.0};
            if (t < dim) {
                T acc = T(0), anti = T(0);
                if (partners) {
#pragma unroll 4
                    for (int b = 0; b < n_bonds; ++b) {
                        const uint32_t i = rows[uint32_t(b) * stride + t];
                        const bool on = i != kNoPartner;
                        const T c = on ? bond_coef<T>(B, b) : T(0), v = x[on ? i : 0u];
                        acc += c * (on ? v : T(0));
                        anti += c;
                    }
                } else {
                    LdsGather<T> vis{x, dim - 1, B, acc, anti};
                    cr_bonds<L, false>(t, L(0), S.n_up, B, C, ylds, vis);
                }
                const T diag = jsum4 - anti, xt = x[t];
                T out = diag * xt + acc;
                out = ab[0] * out - ab[1] * (step == 1 ? T(0) : y[t]);
                prod[0] = double(xt) * double(out);
                y[t] = out;
            }
            wave_fold_columns<1, false>(prod, psum + g);
        }
        __syncthreads();
        if (wave == 0) {
            total();
            if (lane == 0) chain_set_alpha(&chain, tot);
        }
        __syncthreads();
        const T up = sizeof(T) == 4 ? T(chain.up_f) : T(chain.up_d);
        for (uint32_t g = wave; g < groups; g += kTinyThreads / 64) {
            const uint32_t t = g * 64u + uint32_t(lane);
            double part[1] = {0.0};
            if (t < dim) {
                const T v = y[t] - up * x[t];
                part[0] += double(v) * double(v);
                y[t] = v;
            }
            wave_fold_columns<1, false>(part, psum + g);
        }
        __syncthreads();
        if (wave == 0) {
            total();
            if (lane == 0 && finish_beta(&chain, sw, col, step, tot, a.eps)) atomicSub(&sw.state[1], 1);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) sw.chains[col] = chain;
}

// Zeroes every sector's chain states and ticket and sets its step counter to
// 1 with no active chains (one block per sector).
__global__ void chain_init_kernel(LanczosLaunch a) {
    if (blockIdx.x == 0 && a.queue && threadIdx.x < unsigned(kQueueWords)) a.queue[threadIdx.x] = 0u;
    if (int(blockIdx.x) >= a.nsec) return;
    const SecWork& sw = a.secs[blockIdx.x];
    for (int i = threadIdx.x; i < int(a.ld); i += blockDim.x) {
        Chain c{};
        sw.chains[i] = c;
    }
    if (threadIdx.x == 0) {
        *sw.ticket = 0u;
        sw.state[0] = 1;
        sw.state[1] = 0;
    }
}

}  // namespace

hipError_t launch_start(const LanczosLaunch& a, hipStream_t st) {
    const dim3 g(unsigned(a.grid)), b(kBlock);
    if (a.vb < 1 || a.vb > 8) return hipErrorInvalidValue;
    if (a.vb > 4) {
        if (a.dtype == 0) hipLaunchKernelGGL((start_kernel<float, 8>), g, b, 0, st, a);
        else hipLaunchKernelGGL((start_kernel<double, 8>), g, b, 0, st, a);
        return hipGetLastError();
    }
    if (a.dtype == 0) hipLaunchKernelGGL((start_kernel<float, 4>), g, b, 0, st, a);
    else hipLaunchKernelGGL((start_kernel<double, 4>), g, b, 0, st, a);
    return hipGetLastError();
}

hipError_t launch_update(const LanczosLaunch& a, hipStream_t st) {
    const dim3 g(unsigned(a.grid)), b(kBlock);
    auto go = [&](auto tt) {
        using T = decltype(tt);
        return with_vb<T>(a.vb, [&](auto vb) {
            hipLaunchKernelGGL((update_kernel<T, decltype(vb)::value>), g, b, 0, st, a);
            return hipGetLastError();
        });
    };
    return a.dtype == 0 ? go(float{}) : go(double{});
}

hipError_t launch_chain_init(const LanczosLaunch& a, hipStream_t st) {
    hipLaunchKernelGGL(chain_init_kernel, dim3(unsigned(a.nsec)), dim3(64), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_tiny_chains(const LanczosLaunch& a, const ChainBlocks& blocks, int n_bonds, hipStream_t st) {
    size_t lds = tiny_chain_lds(a.max_dim, a.n_sites, a.dtype == 0 ? 4 : 8);
    const size_t rows = tiny_partner_lds(a.max_dim, n_bonds);
    const int partners = lds + rows <= kTinyLds ? 1 : 0;
    if (partners) lds += rows;
    auto go = [&](auto kern) {
        hipError_t e = hipSuccess;
        if (lds > 65536)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    int(lds));
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(unsigned(a.ld), unsigned(a.nsec)), dim3(kTinyThreads), lds, st, a, blocks,
                           partners);
        return hipGetLastError();
    };
    if (a.n_sites > 32) return a.dtype == 0 ? go(tiny_chain_kernel<uint64_t, float>) : go(tiny_chain_kernel<uint64_t, double>);
    return a.dtype == 0 ? go(tiny_chain_kernel<uint32_t, float>) : go(tiny_chain_kernel<uint32_t, double>);
}

bool by_tiny_chains(const LanczosLaunch& a) {
    return a.two_s <= 1 && a.max_dim <= uint64_t(kTinyTiles) * kBlock &&
           tiny_chain_lds(a.max_dim, a.n_sites, a.dtype == 0 ? 4 : 8) <= kTinyLds;
}

}  // namespace ftlm
