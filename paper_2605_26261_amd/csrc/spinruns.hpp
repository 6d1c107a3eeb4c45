// H.x rows by runs at general spin: the scheme of runs.hpp over digit strings
// (spin.hpp). A wave works on rows of one run, whose high sites share their
// digits: which ladder terms between high sites exist, their weights and where
// the partner run of every term begins are found once, one lane per site or
// term. A row's partner in that run is the rank of the changed low string.
#pragma once

#include "runs.hpp"
#include "spin.hpp"
#include "spinlow.hpp"

namespace ftlm {

static __device__ const SpinLowTable<3> kSpinLow3 = make_spin_low_table<3>();
static __device__ const SpinLowTable<4> kSpinLow4 = make_spin_low_table<4>();
static __device__ const SpinLowTable<5> kSpinLow5 = make_spin_low_table<5>();
static __device__ const SpinLowTable<6> kSpinLow6 = make_spin_low_table<6>();

// The low part of a sector with d <= 6: its tables and sites.
struct SpinLow {
    const uint16_t* rank;
    const uint32_t* digits;
    const uint32_t* first;
    int sites, d;
};
template <typename Table>
__device__ __forceinline__ SpinLow spin_low_of(const Table& t, int d) {
    return SpinLow{t.rank, t.digits, t.first, Table::sites, d};
}
__device__ __forceinline__ SpinLow spin_low(const SectorDev& S) {
    switch (S.two_s) {
        case 2: return spin_low_of(kSpinLow3, 3);
        case 3: return spin_low_of(kSpinLow4, 4);
        case 4: return spin_low_of(kSpinLow5, 5);
        default: return spin_low_of(kSpinLow6, 6);
    }
}
__host__ __device__ inline uint32_t spin_low_strings(int d) {
    uint32_t n = 1;
    for (int i = 0; i < spin_low_sites(d); ++i) n *= uint32_t(d);
    return n;
}

// LDS: the ranks of the low strings, then the cumulative dimension table from
// the lowest high site up.
__host__ __device__ inline size_t spin_runs_rank_bytes(const SectorDev& s) {
    return (size_t(spin_low_strings(s.two_s + 1)) * 2 + 15) & ~size_t(15);
}
inline size_t spin_runs_lds(const SectorDev& s) {
    const int high = s.n_sites - spin_low_sites(s.two_s + 1);
    return spin_runs_rank_bytes(s) + size_t(high) * size_t(s.bw) * size_t(s.two_s + 1) * 4;
}

// Digit pairs (a_lo, a_hi) of a bond: {factor of e = +1, of e = -1 (zero where
// the term does not exist), m_lo m_hi, 0} at 4 (8 a_lo + a_hi).
template <typename T>
struct PairTable {
    T v[64 * 4];
    __device__ __forceinline__ void stage(int two_s) {
        if (threadIdx.x >= 64) return;
        const int al = int(threadIdx.x) >> 3, ah = int(threadIdx.x) & 7;
        const double s = 0.5 * two_s;
        auto fu = [&](int a) {  // the ladder factors of spin_lds_setup
            const double m = double(a) - s, q = s * (s + 1.0) - m * (m + 1.0);
            return T((a >= 0 && a <= two_s && q > 0.0) ? sqrt(q) : 0.0);
        };
        const bool in = al <= two_s && ah <= two_s;
        T* e = v + 4 * threadIdx.x;
        e[0] = in && ah > 0 ? fu(al) * fu(ah - 1) : T(0);
        e[1] = in && al > 0 ? fu(al - 1) * fu(ah) : T(0);
        const T st = T(0.5) * T(two_s);
        e[2] = (T(al) - st) * (T(ah) - st);
        e[3] = T(0);
    }
};

// D_c of Eq. (16) for the sites from `site0` up (CumDim without the low sites).
struct HighDim {
    const uint32_t* t;
    int bw, d, site0;
    __device__ __forceinline__ uint32_t operator()(int p, int A, int a) const {
        return t[((p - site0) * bw + A + 1) * d + a];
    }
};

// What a run's high sites decide.
struct SpinRun {
    uint64_t h;      // the high sites' digits, four bits each, from the lowest one up
    uint32_t base;   // the run's first row
    uint32_t size;   // its rows
    int k;           // digit sum of the low sites
    uint32_t xp, xm, yp, ym;  // lane i: X_e, Y_e (spin_cr_row) of site N - 1 - i
    uint32_t tp, tm;          // sum of T_e over the high sites

    __device__ __forceinline__ void find(uint32_t row, const SectorDev& S, HighDim D, int low, int lane) {
        lane = opaque(lane);
        const int N = S.n_sites, nh = N - low;
        uint32_t rem = row;
        int A = S.n_up, my_A = 0, my_a = 0;
        h = 0;
        for (int q = N - 1; q >= low; --q) {
            const uint32_t c = D(q, A, lane <= S.two_s ? lane : 0);
            const int a = 63 - __builtin_clzll(__ballot(lane <= S.two_s && c <= rem));
            if (lane == N - 1 - q) {
                my_A = A;
                my_a = a;
            }
            rem -= lane_u32(c, a);
            A -= a;
            h = (h << 4) | uint64_t(uint32_t(a));
        }
        base = row - rem;
        k = A;
        size = uniform(D(low, A, 1));
        size = size ? size : 1u;  // never: the run holds `row`; a walk over runs always moves on
        const bool on = lane < nh;
        const int q = on ? N - 1 - lane : N - 1;
        if (!on) my_A = my_a = 0;
        const uint32_t c0 = D(q, my_A, my_a);
        const uint32_t Tp = on ? D(q, my_A + 1, my_a) - c0 : 0u, Tm = on ? D(q, my_A - 1, my_a) - c0 : 0u;
        const uint32_t Pp = wave_prefix_sum(Tp), Pm = wave_prefix_sum(Tm);
        tp = lane_u32(Pp, 63);
        tm = lane_u32(Pm, 63);
        const bool up = my_a < S.two_s, dn = my_a > 0;
        const int au = up ? my_a + 1 : my_a, ad = dn ? my_a - 1 : my_a;
        xp = (up ? D(q, my_A + 1, au) : 0u) - c0 + (Pp - Tp);
        xm = (dn ? D(q, my_A - 1, ad) : 0u) - c0 + (Pm - Tm);
        yp = (dn ? D(q, my_A, ad) : 0u) - c0 - Pp;
        ym = (up ? D(q, my_A, au) : 0u) - c0 - Pm;
    }
};

// Up to kSpinSetBonds bonds of a run: lane 2 i holds term e = +1 of bond i, lane
// 2 i + 1 its term e = -1. Lanes 62 and 63 hold none.
constexpr int kSpinSetBonds = 31;
constexpr int kNoTerm = 63;

template <typename T>
struct SpinTerms {
    uint32_t blo, bhi;  // address of the first row of the run that the term's partners lie in
    T coef;             // J_b / 2
    T w;                // between high sites: the term's weight
    uint32_t digits;    // a bond with a low site: shifts of its digits in the low string (bits 0, 8), width of the
                        // higher one's (bit 16; zero when that site is high) and the high one's digit (bit 24)
    int step;           // what e = +1 adds to the low string
    uint64_t flips;     // the terms between high sites that exist; bit kNoTerm is always set
    T dsum;             // diagonal sum of the bonds between high sites, these and the sets before

    __device__ __forceinline__ void load(const SpinRun& run, const SectorDev& S, const BondTable& B, const T* pairs,
                                         int first, int low, int lane, const unsigned char* xb, uint32_t ldb) {
        lane = opaque(lane);
        const int b = first + (lane >> 1), N = S.n_sites, d = S.two_s + 1;
        const bool minus = (lane & 1) != 0, on = lane < 2 * kSpinSetBonds && b < B.n_bonds;
        const uint32_t pack = on ? B.pack[b] : 0u;
        coef = on ? bond_coef<T>(B, b) : T(0);
        const int lo = int(pack & 0xffu), hi = int((pack >> 8) & 0xffu);
        const bool in_low = lo < low, cross = in_low && hi >= low;
        const uint32_t x_p = uint32_t(__builtin_amdgcn_ds_bpermute((N - 1 - lo) * 4, int(run.xp)));
        const uint32_t x_m = uint32_t(__builtin_amdgcn_ds_bpermute((N - 1 - lo) * 4, int(run.xm)));
        const uint32_t y_p = uint32_t(__builtin_amdgcn_ds_bpermute((N - 1 - hi) * 4, int(run.yp)));
        const uint32_t y_m = uint32_t(__builtin_amdgcn_ds_bpermute((N - 1 - hi) * 4, int(run.ym)));
        const uint32_t x = minus ? x_m : x_p, y = minus ? y_m : y_p;
        uint32_t tgt = run.base + (cross ? y + (minus ? run.tm : run.tp) : in_low ? 0u : x + y);
        tgt = tgt < S.dim - 1 ? tgt : S.dim - 1;  // of a term that no row has; nothing is read from it
        const uint64_t at = reinterpret_cast<uint64_t>(xb) + uint64_t(tgt) * ldb;
        blo = uint32_t(at);
        bhi = uint32_t(at >> 32) & 0xffffu;
        const int al = in_low ? 0 : int((run.h >> (4 * (lo - low))) & 15u);
        const int ah = hi >= low ? int((run.h >> (4 * (hi - low))) & 15u) : 0;
        const T* e = pairs + 4 * ((al & 7) * 8 + (ah & 7));
        const T f = minus ? e[1] : e[0];
        const bool high = on && !in_low;
        w = high ? coef * f : T(0);
        flips = __ballot(high && f != T(0)) | (uint64_t(1) << kNoTerm);
        digits = uint32_t(4 * lo) & 31u;
        digits |= hi < low ? uint32_t(4 * hi) << 8 | 4u << 16 : uint32_t(ah) << 24;
        int pl = 1, ph = 1;
        for (int i = 0; i < low; ++i) {
            pl *= i < lo ? d : 1;
            ph *= i < hi ? d : 1;
        }
        step = pl - (hi < low ? ph : 0);
        // the diagonal of the bonds between high sites, in the bonds' order
        const T two = T(2) * coef, mm = e[2];
        if (first == 0) dsum = T(0);
        const int n = __builtin_popcountll(__ballot(high)) / 2;
        for (int i = 0; i < n; ++i) dsum += lane_val(two, 2 * i) * lane_val(mm, 2 * i);
    }
};

// Rows of x of the G terms of a slot and their weights.
template <typename T, int VB, int R, int G>
struct SpinSlot {
    T v[G][R][VB];
    T w[G][R];
};

// y = H x on the rows lo <= t < hi of one run, at most 64 R (lane l: rows lo + l,
// lo + 64 + l, ...), as run_block. Bonds go in the sorted order of the bond
// table, each with its terms e = +1 and -1, one bond a slot, two slots in turn:
// every sum has the terms of spin_cr_row in the same order, with the same
// weights, each fused with its product (left to the compiler, a product that
// ended in another block than its sum was rounded by itself: 3 % of the rows of
// one column differed in the last bit). A row without a term loads nothing for it.
template <typename T, int VB, int R>
__device__ __forceinline__ void spin_run_block(const SectorDev& S, const BondTable& B, const uint16_t* rank,
                                               const SpinLow& L, const T* pairs, const SpinRun& run, SpinTerms<T>& st,
                                               const T* __restrict__ x, T* __restrict__ y, uint64_t ld, uint32_t col0,
                                               uint32_t row0, uint32_t lo, uint32_t hi) {
    constexpr int G = 2;  // terms of a bond
    const int lane = threadIdx.x & 63;
    const uint32_t ldb = uint32_t(ld * sizeof(T));
    const unsigned char* xb = reinterpret_cast<const unsigned char*>(x + col0);
    const uint32_t bytes = uniform(kRunRows * ldb);
    const int n_bonds = uniform(B.n_bonds);
    const int n_high = uniform(int(B.ends[L.sites]));
    const uint32_t* strings = L.digits + uniform(*gptr(L.first + run.k));
    const uint32_t j0 = lo - run.base, jn = hi - lo;
    uint32_t voff[R], dig[R], low[R];
    T acc[R][VB], dsum[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const uint32_t j = j0 + uint32_t(64 * i + lane);
        const bool in = j - j0 < jn;
        voff[i] = in ? __umul24(j, ldb) : kNoRow;
        dig[i] = *gptr(strings + (in ? j : j0));
        low[i] = 0;
        for (int q = L.sites - 1; q >= 0; --q)
            low[i] = __umul24(low[i], uint32_t(L.d)) + __builtin_amdgcn_ubfe(dig[i], uint32_t(4 * q), 4u);
#pragma unroll
        for (int c = 0; c < VB; ++c) acc[i][c] = T(0);
    }
    SpinSlot<T, VB, R, G> sa, sb;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int i = 0; i < R; ++i) {
            sb.w[g][i] = T(0);
#pragma unroll
            for (int k = 0; k < VB; ++k) sb.v[g][i][k] = T(0);
        }
    auto add = [&](auto& sl) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int k = 0; k < VB; ++k) acc[i][k] = fma(sl.w[g][i], sl.v[g][i][k], acc[i][k]);
    };
#pragma unroll
    for (int i = 0; i < R; ++i) dsum[i] = st.dsum;
#pragma unroll 1
    for (int set = 0; set < n_bonds; set += kSpinSetBonds) {
        if (n_bonds > kSpinSetBonds) {
            st.load(run, S, B, pairs, set, L.sites, lane, xb, ldb);
            if (set == 0 || n_high > set) {
#pragma unroll
                for (int i = 0; i < R; ++i) dsum[i] = st.dsum;
            }
        }
        uint64_t fl = st.flips;
        auto high = [&](auto& sl) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int t = __builtin_ctzll(fl);
                fl = (fl & (fl - 1)) | (uint64_t(1) << kNoTerm);
                const T w = lane_val(st.w, t);
                const auto rs = run_rsrc(lane_u32(st.blo, t), lane_u32(st.bhi, t), t < kNoTerm ? bytes : 0u);
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    sl.w[g][i] = w;
                    buffer_row<T, VB>(rs, voff[i], sl.v[g][i]);
                }
            }
        };
        while (fl != uint64_t(1) << kNoTerm) {
            high(sa);
            add(sb);
            high(sb);
            add(sa);
        }
        const int nb = n_bonds - set < kSpinSetBonds ? n_bonds - set : kSpinSetBonds;
        // bond b of the set for rows i: partner offsets and weights of its terms
        uint32_t off[2][R];
        T w[2][R];
        auto prepare = [&](int b) {
            const uint32_t dg = lane_u32(st.digits, 2 * b);
            const int step = int(lane_u32(uint32_t(st.step), 2 * b));
            const T c = lane_val(st.coef, 2 * b);
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const uint32_t al = __builtin_amdgcn_ubfe(dig[i], dg & 31u, 4u);
                const uint32_t ah = __builtin_amdgcn_ubfe(dig[i], (dg >> 8) & 31u, (dg >> 16) & 15u) + (dg >> 24);
                const T* e = pairs + 4 * ((al & 7u) * 8u + (ah & 7u));
                const T f0 = e[0], f1 = e[1], mm = e[2];
                dsum[i] += T(2) * c * mm;
                const uint32_t r0 = rank[int(low[i]) + (f0 != T(0) ? step : 0)];
                const uint32_t r1 = rank[int(low[i]) - (f1 != T(0) ? step : 0)];
                off[0][i] = f0 != T(0) ? __umul24(r0, ldb) : kNoRow;
                off[1][i] = f1 != T(0) ? __umul24(r1, ldb) : kNoRow;
                w[0][i] = c * f0;
                w[1][i] = c * f1;
            }
        };
        auto fetch = [&](auto& sl, int g, int b, int e) {
            const auto rs = run_rsrc(lane_u32(st.blo, 2 * b + e), lane_u32(st.bhi, 2 * b + e), bytes);
#pragma unroll
            for (int i = 0; i < R; ++i) {
                sl.w[g][i] = w[e][i];
                buffer_row<T, VB>(rs, off[e][i], sl.v[g][i]);
            }
        };
        int b = n_high > set ? n_high - set : 0;
        for (; b + 1 < nb; b += 2) {
            prepare(b);
            fetch(sa, 0, b, 0);
            fetch(sa, 1, b, 1);
            add(sb);
            prepare(b + 1);
            fetch(sb, 0, b + 1, 0);
            fetch(sb, 1, b + 1, 1);
            add(sa);
        }
        if (b < nb) {
            prepare(b);
            fetch(sa, 0, b, 0);
            fetch(sa, 1, b, 1);
            add(sb);
            sb = sa;
        }
    }
    add(sb);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const uint32_t j = j0 + uint32_t(64 * i + lane);
        if (j - j0 < jn) {
            const uint32_t t = run.base + j;
            T xt[VB], out[VB];
            load_row<T, VB>(reinterpret_cast<const T*>(xb + uint64_t(t) * ldb), xt);
#pragma unroll
            for (int c = 0; c < VB; ++c) out[c] = dsum[i] * xt[c] + acc[i][c];
            T* yrow = y + uint64_t(t - row0) * ld + col0;
            store_row<T, VB>(yrow, out);
        }
    }
}

// The sector rows [pos, end) by one wave, 64 R rows of a run at a time: y = H x.
template <typename T, int VB, int R>
__device__ __forceinline__ void spin_run_rows(const SectorDev& S, const BondTable& B, const uint16_t* rank, HighDim D,
                                              const SpinLow& L, const T* pairs, const T* __restrict__ x,
                                              T* __restrict__ y, uint64_t ld, uint32_t col0, uint32_t row0,
                                              uint32_t pos, uint32_t end) {
    const int lane = threadIdx.x & 63;
    const unsigned char* xb = reinterpret_cast<const unsigned char*>(x + col0);
    while (pos < end) {
        SpinRun run;
        run.find(pos, S, D, L.sites, lane);
        const uint32_t lim = end - run.base < run.size ? end : run.base + run.size;
        SpinTerms<T> st;
        st.load(run, S, B, pairs, 0, L.sites, lane, xb, uint32_t(ld * sizeof(T)));
#pragma unroll 1
        for (; pos < lim; pos = lim - pos > uint32_t(64 * R) ? pos + uint32_t(64 * R) : lim)
            spin_run_block<T, VB, R>(S, B, rank, L, pairs, run, st, x, y, ld, col0, row0, pos, lim);
    }
}

}  // namespace ftlm
