// Host-side machinery shared by the C ABI (abi.cpp) and the request server
// (server.cpp). Internal to libftlm.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "ftlm.h"
#include "host_math.hpp"
#include "kernels.hpp"

struct ftlm_graph {
    int n_sites = 0;
    std::vector<int> bi, bj;   // merged bonds, caller order of first appearance
    std::vector<double> J;
    int n_input = 0;           // bonds as given (before merging)
    std::vector<int> merged_of_input;
    ftlm::BondTable table{};   // in the caller's site labels
};

struct ftlm_sector {
    int n_sites = 0, n_up = 0, mode = 0;
    int two_s = 1;          // 2s of the local spin; n_up is the digit sum A when two_s > 1
    uint64_t dim = 0;
    void* table = nullptr;
    size_t bytes = 0;
    ftlm::TableLayout layout{};
    std::vector<uint32_t> binom_host;
    ftlm::SectorDev dev{};
};

namespace ftlm {

// Thread-local error text behind ftlm_last_error; fail() records a message and
// returns its code, ok() clears it.
extern thread_local std::string g_err;
int fail(int code, const char* fmt, ...);
int ok();

#define HIP_CHECK(expr)                                                                                \
    do {                                                                                               \
        hipError_t e_ = (expr);                                                                        \
        if (e_ != hipSuccess) return ::ftlm::fail(FTLM_E_DEVICE, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

uint64_t binom_u64(int n, int k);

// Weight of a sector in the thermal sums: the sectors +M and -M have the
// same spectrum (Sec. 2), so a sector with M != 0 stands for both.
inline double sector_multiplicity(int n_sites, int n_up) { return 2 * n_up == n_sites ? 1.0 : 2.0; }

// Two timing events destroyed on every exit path.
struct EventPair {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t create() {
        hipError_t e = hipEventCreate(&e0);
        return e == hipSuccess ? hipEventCreate(&e1) : e;
    }
    EventPair() = default;
    EventPair(const EventPair&) = delete;
    EventPair& operator=(const EventPair&) = delete;
    ~EventPair() {
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
    }
};

// Bond tables of the row kernels (bonds.cpp).
BondTable make_bond_table(int n_sites, const std::vector<int>& lo, const std::vector<int>& hi,
                          const std::vector<double>& J, const std::vector<int>& orig, double jsum_all);
constexpr int kTablesPerGraph = 1;  // the graph's bond table
uint64_t stream_key(uint64_t seed, int n_up, uint64_t r);

// ---- stats -------------------------------------------------------------------
struct Stats {
    std::mutex mu;
    bool on = false;
    int64_t launches = 0;
    double ms = 0.0;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> pending;
};
extern Stats g_stats;

struct HvTimer {
    hipEvent_t a = nullptr, b = nullptr;
    hipStream_t st;
    static bool wanted() {
        std::lock_guard<std::mutex> lk(g_stats.mu);
        return g_stats.on;
    }
    explicit HvTimer(hipStream_t s) : st(s) {
        std::lock_guard<std::mutex> lk(g_stats.mu);
        if (!g_stats.on) return;
        if (hipEventCreate(&a) != hipSuccess) {
            a = nullptr;
            return;
        }
        if (hipEventCreate(&b) != hipSuccess) {
            (void)hipEventDestroy(a);
            a = b = nullptr;
            return;
        }
        (void)hipEventRecord(a, st);
    }
    ~HvTimer() {
        if (!a) return;
        (void)hipEventRecord(b, st);
        std::lock_guard<std::mutex> lk(g_stats.mu);
        g_stats.pending.emplace_back(a, b);
    }
};

std::vector<std::pair<int, int>> column_chunks(int nvec, int dtype, int max_width, bool blocks = false,
                                               const std::vector<const void*>& ptrs = {});
// Widest launch of the H.x kernels of a sector: 8 columns for general spin.
inline int max_launch_width(int two_s) { return two_s > 1 ? 8 : 32; }
// Columns of a Lanczos launch at most. Large sectors are bound by the partner
// lines that miss L2, of which up to eight columns move the fewest per column (by runs
// from 2^26 rows); small ones by the launches. The line goes by the sites
// alone, so that requests of one size run together whatever their sectors. 32
// FP32 columns, a step, half filling, at most 32 / 20 or 16 / 8 columns a launch:
// 18 sites 55 / 76 / 111 us, 20 sites 133 / 130 / 163, 21 sites 236 / 208 / 239, 22
// sites 394 / 357 / 365, 24 sites 1385 / 1212 / 1116, 26 sites 6321 / 5368 / 4973; 20
// columns at 21 sites 119 in one launch, 148 as 16 and 4. 16 FP64 columns, 16 / 8:
// 18 sites 65 / 78, 20 sites 177 / 148, 24 sites 1362 / 1156. A sector of many
// sites with few spins up is smaller than its sites say, and takes more launches
// than one of its size would (24 sites, 21 up, 2,024 rows, 32 columns 100 us a step
// in four launches). From 36 sites on sectors within reach have few spins up, or down:
// few partners to load, but many sites to rank. Up to 20 columns take one launch (20
// in one / 8, 8 and 4: 36 sites, 7 down 2.61 / 3.01 ms, 10 up 99.8 / 95.1 with cluster
// bonds, 90.8 / 92.5 on a ring, 40, 7 down 5.97 / 6.61, 52, 6 down 8.51 / 11.4; but 34,
// 10 up 56.5 / 53.8, 33, 12 up 155 / 143); more of them 16 or 32 from 42 sites (32 in
// one / 8 a launch: 40, 7 down 10.2 / 9.4, 42, 6 down 3.18 / 4.01, 52, 6 down 12.1 /
// 15.7; 24 as 20 and 4 / 16 and 8 / 8 a launch: 44, 6 down 4.31 / 4.17 / 4.09 with
// cluster bonds, 3.90 / 3.70 / 3.98 on a ring). FP64, 16 in one / 8 a launch: 47 sites,
// 6 down 5.83 / 5.66 and 6.11 / 6.30, 52, 6 down 11.6 / 11.5 and 12.0 / 12.5.
inline int lanczos_width(int two_s, int n_sites, int dtype, int R) {
    if (two_s > 1) return max_launch_width(two_s);
    if (dtype != FTLM_F32) return n_sites <= 18 || n_sites >= 52 ? 16 : 8;
    if (n_sites >= 36 && R <= 20) return 20;
    if (n_sites >= 42) return R >= 32 ? 32 : 16;
    return n_sites <= 20 ? 32 : n_sites <= 22 ? 20 : 8;
}
int check_dtype(int dtype);

// Byte offsets of one sector's Lanczos state inside a workspace or arena.
struct SectorState {
    size_t u0, u1, partials, chains, alpha, beta, ticket, keys, state;
};
size_t partial_bytes(uint64_t dim, int R, int dtype);
size_t layout_state(uint64_t dim, int R, int dtype, size_t off, SectorState& st);

template <typename P>
P* at(void* base, size_t off) { return reinterpret_cast<P*>(static_cast<char*>(base) + off); }

// A batch of R chains in each of a list of sectors (one sector for
// ftlm_lanczos, all sectors of a plan), with the device descriptors of the
// multi-sector Lanczos kernels. Host copies stay alive until the stream work
// that reads them has been synchronized.
struct LanczosJob {
    int nsec = 0, R = 0, dtype = 0, mode = 0, n_sites = 0, grid = 0, two_s = 1;
    int items = 0;                       // work items of the persistent H.x, all sectors
    size_t lds = 0;
    std::vector<SecWork> secs;           // host copies of the descriptors
    std::vector<uint64_t> keys;          // [nsec][R] stream keys of the run
    SecWork* dev_secs = nullptr;
    std::vector<uint64_t*> key_ptrs;
    std::vector<BondTable> bonds;        // host copies, one per distinct device table
    std::vector<BondTable*> dev_bonds;   // where each copy goes
    std::vector<std::pair<int, int>> chunks;
    int max_steps = 0;                   // largest m_eff over the sectors
    uint32_t* queue = nullptr;           // work-queue counters of the persistent H.x (kQueueBytes)

    LanczosLaunch launch() const {
        LanczosLaunch a{};
        a.secs = dev_secs;
        a.nsec = nsec;
        a.grid = grid;
        a.items = items;
        for (const SecWork& w : secs) {
            a.max_dim = std::max<uint64_t>(a.max_dim, w.S.dim);
            a.max_bw = std::max(a.max_bw, w.S.bw);
            a.xcd_items += int(xcd_items(w.items, 0));
            a.xcd_pairs += int(xcd_items((w.items + 1) / 2, 0));
        }
        a.n_up = secs.empty() ? 0 : secs[0].S.n_up;
        a.ld = uint64_t(R);
        a.dtype = dtype;
        // FP32 vectors: an exact invariant subspace leaves a residual of about
        // 1e-5 of the coefficient scale (FP32 row sums and vector updates), so
        // the threshold sits a factor 10 above it
        a.eps = dtype == FTLM_F32 ? 1e-4 : 1e-12;
        a.mode = mode;
        a.n_sites = n_sites;
        a.two_s = two_s;
        a.queue = queue;
        return a;
    }
};

// Sector i runs with graph graphs[graph_of[i]] (null: no H.x, start vectors
// only), whose kTablesPerGraph bond tables go to dev_tables[graph_of[i]].
void job_layout(LanczosJob& job, const std::vector<SectorDev>& devs, const std::vector<SectorState>& states,
                void* base, int R, int M, int dtype, SecWork* dev_secs, const std::vector<const ftlm_graph*>& graphs,
                const std::vector<BondTable*>& dev_tables, const std::vector<int>& graph_of);
int job_start(LanczosJob& job, uint64_t seed, uint64_t r0, int dist, hipStream_t st);
// The job's columns split into launches of at most max_width columns.
std::vector<std::pair<int, int>> job_chunks(const LanczosJob& job, int max_width);
int job_steps(const LanczosJob& job, hipStream_t st, bool timed = true, int nsteps = -1);
int job_collect(const LanczosJob& job, int M, double* alpha_host, double* beta_host, int32_t* steps_host,
                hipStream_t st);

}  // namespace ftlm
