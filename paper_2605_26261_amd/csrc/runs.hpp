// H.x rows by runs (spin 1/2).
//
// The rows whose labels share every site from kLowBits up form a run of
// consecutive sector rows: the low sites take all patterns with the remaining
// up spins, in ascending order. A wave works on rows of one run at a time, so
// all that depends on the high sites is the same for its 64 lanes and is
// computed once, one lane per site or bond: which bonds between high sites
// flip, and where the partner run of every bond begins. Inside a run the
// partner's position is the rank of the flipped low pattern, one LDS read.
#pragma once

#include "lowtab.hpp"
#include "rowio.hpp"
#include "rowloop.hpp"

namespace ftlm {

static __device__ const LowTables kLow = make_low_tables();

__device__ __forceinline__ uint32_t lane_u32(uint32_t v, int lane) {
    return uint32_t(__builtin_amdgcn_readlane(int(v), lane));
}
__device__ __forceinline__ float lane_val(float v, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ double lane_val(double v, int lane) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint64_t lo = lane_u32(uint32_t(u), lane), hi = lane_u32(uint32_t(u >> 32), lane);
    return __builtin_bit_cast(double, lo | (hi << 32));
}

// The same value, as the compiler cannot know: what is computed from it stays
// where it is used. (Hoisted out of the loop over the items, the lane's part of
// find() and load() held 80 registers through the bond loops.)
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Inclusive prefix sum over the lanes of a wave (every lane active).
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t v) {
    int x = int(v);
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
    return uint32_t(x);
}

// Bonds handled together, one per lane; lane kSetBonds holds none.
constexpr int kSetBonds = 63;

// What a run's high sites decide, found by all lanes of a wave together.
template <typename L>
struct Run {
    L h;             // the high sites' pattern
    uint32_t base;   // the run's first row
    uint32_t size;   // its rows
    int k;           // up spins among the low sites
    uint32_t X, Y, Z;  // lane i: the terms of site N - 1 - i in the partners' first rows

    __device__ __forceinline__ void find(uint32_t row, const SectorDev& S, Binom C, int low_bits, int lane) {
        lane = opaque(lane);
        const int N = S.n_sites;
        uint32_t rem = row;
        int A = S.n_up;
        h = 0;
        // six sites at a time: lane i counts the rows below pattern i of the
        // six, the run's pattern is the last one that begins at or before `row`
        for (int top = N; top > low_bits;) {
            const int n = top - low_bits < 6 ? top - low_bits : 6;
            uint32_t below = 0;
            int a = A;
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                const int q = top - 1 - i;                      // the site; its bit in the lane index is n - 1 - i
                const bool one = i < n && (((lane << i) >> (n - 1)) & 1);
                const uint32_t c = C(i < n ? q : 0, a > 0 ? a : 0);
                below += one ? c : 0u;
                a -= one ? 1 : 0;
            }
            // a >= 0 up spins are left for the sites below; with more than
            // there are sites the pattern has no rows and begins where the next one does
            const uint64_t ok = __ballot(lane < (1 << n) && a >= 0 && below <= rem);
            const int pat = 63 - __builtin_clzll(ok);
            rem -= lane_u32(below, pat);
            A -= __popc(uint32_t(pat));
            h = (h << n) | L(pat);
            top -= n;
        }
        base = row - rem;
        k = A;
        size = low_bits < N ? uint32_t(__builtin_amdgcn_readfirstlane(int(C(low_bits, A)))) : S.dim;
        size = size ? size : 1u;  // never: the run holds `row`; a walk over runs always moves on
        // lane i holds site q = N - 1 - i (the formulas of cr_bonds)
        const int nh = N - low_bits;
        {
            const bool on = lane < nh;
            const int q = on ? N - 1 - lane : N - 1;
            const L up = nh > 0 ? h >> (q - low_bits) : L(0);
            const bool bit = on && (up & 1) != 0;
            const int K = S.n_up - popc(L(L(up) >> 1));
            const uint32_t cm = C(q, K - 1), c0 = C(q, K), cp = C(q, K + 1);
            const uint32_t d1 = bit ? cm - c0 : 0u, d2 = bit ? cp - c0 : 0u;
            const uint32_t P1 = wave_prefix_sum(d1), P2 = wave_prefix_sum(d2);
            const uint32_t t1 = lane_u32(P1, 63), t2 = lane_u32(P2, 63);
            X = bit ? P1 - d1 - c0 : cp + P2;
            Y = bit ? 0u - cp - (P2 - d2) : c0 - P1;
            Z = bit ? t2 - P2 - c0 : c0 + t1 - P1;
        }
    }
};

// Up to kSetBonds bonds of a run, one per lane.
template <typename T>
struct RunBonds {
    uint32_t blo, bhi;  // address of the first row of the run that the bond's partners lie in
    uint32_t mask;      // low sites that the bond flips (byte offsets into the rank table: pattern * 2);
                        // bit 30: added to the number of them that are up, it makes an even sum in the rows that flip
    T coef;
    uint64_t flips;     // the bonds between high sites that flip; bit kSetBonds is always set

    template <typename L>
    __device__ __forceinline__ void load(const Run<L>& run, const BondTable& B, int first, int low_bits, int lane,
                                         const unsigned char* xb, uint32_t ldb, uint32_t last) {
        lane = opaque(lane);
        const int b = first + lane, N = B.n_sites;
        const bool on = lane < kSetBonds && b < B.n_bonds;
        const uint32_t pack = on ? B.pack[b] : 0u;
        coef = on ? bond_coef<T>(B, b) : T(0);
        const int lo = int(pack & 0xffu), hi = int((pack >> 8) & 0xffu);
        const bool low = lo < low_bits, cross = low && hi >= low_bits;
        const int al = low ? 0 : lo - low_bits, ah = hi >= low_bits ? hi - low_bits : 0;
        const uint32_t uh = uint32_t((run.h >> ah) & 1), ul = uint32_t((run.h >> al) & 1);
        const uint32_t x = uint32_t(__builtin_amdgcn_ds_bpermute((N - 1 - lo) * 4, int(run.X)));
        const uint32_t y = uint32_t(__builtin_amdgcn_ds_bpermute((N - 1 - hi) * 4, int(run.Y)));
        const uint32_t z = uint32_t(__builtin_amdgcn_ds_bpermute((N - 1 - hi) * 4, int(run.Z)));
        uint32_t tgt = run.base + (cross ? z : low ? 0u : x + y);
        tgt = tgt < last ? tgt : last;  // a run without rows may begin past the end; nothing is read from it
        const uint64_t at = reinterpret_cast<uint64_t>(xb) + uint64_t(tgt) * ldb;
        blo = uint32_t(at);
        bhi = uint32_t(at >> 32) & 0xffffu;
        // a low-low bond flips when one of its sites is up, a cross bond when
        // its low site differs from its high one, no bond never
        mask = on && low ? (2u << lo) | (cross ? 0u : 2u << hi) : 0u;
        mask |= (on && cross ? 1u - uh : 1u) << 30;
        flips = __ballot(on && !low && ul != uh) | (uint64_t(1) << kSetBonds);
    }
};

constexpr uint32_t kNoRow = 0x80000000u;  // a byte offset past every buffer: loads return 0 and touch nothing

// Rows of a run at most (C(14, 7) = 3432; general spin 1107). A bond's buffer
// begins at a row of x, where its partners' run begins, and ends after this many:
// a defect in the ranks would read a run's length past x at most. (The rest of x
// as each bond's end cost one column 2 to 5 %.)
constexpr uint32_t kRunRows = 3432;

// A buffer of `bytes` bytes at address hi:lo.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t run_rsrc(uint32_t lo, uint32_t hi, uint32_t bytes) {
    void* p = reinterpret_cast<void*>(uint64_t(lo) | (uint64_t(hi) << 32));
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, int(bytes), kBufferWord3);
}

// VB values at byte offset `off` of a buffer (4-byte aligned).
template <typename T, int VB>
__device__ __forceinline__ void buffer_row(__amdgpu_buffer_rsrc_t rs, uint32_t off, T (&v)[VB]) {
    constexpr int kBytes = VB * int(sizeof(T));
    typedef uint32_t U2 __attribute__((ext_vector_type(2)));
    typedef uint32_t U4 __attribute__((ext_vector_type(4)));
    uint32_t w[kBytes / 4];
    if constexpr (kBytes % 16 == 0) {
#pragma unroll
        for (int k = 0; k < kBytes / 16; ++k) {
            const U4 q = __builtin_amdgcn_raw_buffer_load_b128(rs, int(off + 16 * k), 0, 0);
            w[4 * k] = q.x; w[4 * k + 1] = q.y; w[4 * k + 2] = q.z; w[4 * k + 3] = q.w;
        }
    } else if constexpr (kBytes % 8 == 0) {
#pragma unroll
        for (int k = 0; k < kBytes / 8; ++k) {
            const U2 q = __builtin_amdgcn_raw_buffer_load_b64(rs, int(off + 8 * k), 0, 0);
            w[2 * k] = q.x; w[2 * k + 1] = q.y;
        }
    } else {
#pragma unroll
        for (int k = 0; k < kBytes / 4; ++k) w[k] = __builtin_amdgcn_raw_buffer_load_b32(rs, int(off + 4 * k), 0, 0);
    }
#pragma unroll
    for (int c = 0; c < VB; ++c) {
        if constexpr (sizeof(T) == 4) v[c] = __builtin_bit_cast(T, w[c]);
        else v[c] = __builtin_bit_cast(T, uint64_t(w[2 * c]) | (uint64_t(w[2 * c + 1]) << 32));
    }
}

// Rows of x of G bonds and their weights J_b / 2.
template <typename T, int VB, int R, int G>
struct RunSlot {
    T v[G][R][VB];
    T c[G];
};

// The rows lo <= t < hi of one run among the 64 R rows that begin at row p0
// (lane l: rows p0 + l, p0 + 64 + l, ...): y = H x, or the Lanczos epilogue w =
// hv_a (H u_k) - hv_b u_{k-1} of hv_body, whose products u_k[t] w[t] go to
// prod (zero for the block's other rows). y holds sector row
// `row0` at its start; `low` is the rank table in LDS. Bonds go in the sorted
// order of the bond table, G at a time into two slots in turn: a slot's rows
// are added to the sums after the other slot's loads are issued. Those between
// high sites come first and only where they flip; a row whose bond does not
// flip loads nothing (an offset past the buffer gives 0). Every sum has the
// terms of the row-by-row kernel in the same order.
template <typename L, typename T, int VB, int R, int G, int EPI>
__device__ __forceinline__ void run_block(const SectorDev& S, const BondTable& B, const unsigned char* low,
                                          int low_bits, const Run<L>& run, RunBonds<T>& rb,
                                          const T* __restrict__ x, T* __restrict__ y, uint64_t ld, uint32_t col0,
                                          uint32_t row0, uint32_t p0, uint32_t lo, uint32_t hi, const T* ab,
                                          bool first, double (&prod)[R][VB]) {
    const int lane = threadIdx.x & 63;
    const uint32_t ldb = uint32_t(ld * sizeof(T));
    const unsigned char* xb = reinterpret_cast<const unsigned char*>(x + col0);
    const int n_bonds = __builtin_amdgcn_readfirstlane(B.n_bonds);
    const int n_high = __builtin_amdgcn_readfirstlane(int(B.ends[low_bits]));
    const uint32_t bytes = uniform(kRunRows * ldb);
    const T jsum4 = sizeof(T) == 4 ? T(B.jsum4_f) : T(B.jsum4_d);
    const uint16_t* pat = kLow.pattern + kLow.first[run.k];
    // rows by their position in the run (p0 may lie before it)
    const uint32_t j0 = p0 - run.base, jlo = lo - run.base, jn = hi - lo;
    uint32_t voff[R], l2[R];
    T acc[R][VB], anti[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const uint32_t j = j0 + uint32_t(64 * i + lane);
        const bool in = j - jlo < jn;
        voff[i] = in ? __umul24(j, ldb) : kNoRow;
        l2[i] = 2u * uint32_t(*gptr(pat + (in ? j : jlo)));
        anti[i] = T(0);
#pragma unroll
        for (int c = 0; c < VB; ++c) acc[i][c] = T(0);
    }
    T ah = T(0);
    RunSlot<T, VB, R, G> sa, sb;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        sb.c[g] = T(0);
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int k = 0; k < VB; ++k) sb.v[g][i][k] = T(0);
    }
    auto add = [&](auto& sl) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int k = 0; k < VB; ++k) acc[i][k] += sl.c[g] * sl.v[g][i][k];
    };
#pragma unroll 1
    for (int set = 0; set < n_bonds; set += kSetBonds) {
        if (n_bonds > kSetBonds) rb.load(run, B, set, low_bits, lane, xb, ldb, S.dim - 1);
        uint64_t fl = rb.flips;
        auto high = [&](auto& sl) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int b = __builtin_ctzll(fl);
                fl = (fl & (fl - 1)) | (uint64_t(1) << kSetBonds);
                sl.c[g] = lane_val(rb.coef, b);
                const auto rs = run_rsrc(lane_u32(rb.blo, b), lane_u32(rb.bhi, b), b < kSetBonds ? bytes : 0u);
#pragma unroll
                for (int i = 0; i < R; ++i) buffer_row<T, VB>(rs, voff[i], sl.v[g][i]);
                ah += sl.c[g];
            }
        };
        int b = n_high > set ? n_high - set : 0;
        auto lows = [&](auto& sl) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int bb = b + g < kSetBonds ? b + g : kSetBonds;
                const uint32_t pm = lane_u32(rb.mask, bb);
                const uint32_t mask = pm & 0x3fffffffu, odd = pm >> 30;
                sl.c[g] = lane_val(rb.coef, bb);
                const auto rs = run_rsrc(lane_u32(rb.blo, bb), lane_u32(rb.bhi, bb), bytes);
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const uint32_t no = (uint32_t(__popc(l2[i] & mask)) + odd) << 31;  // kNoRow unless the row flips
                    const uint32_t rank = *reinterpret_cast<const uint16_t*>(low + (l2[i] ^ mask));
                    buffer_row<T, VB>(rs, __umul24(rank, ldb) + no, sl.v[g][i]);
                    anti[i] += no ? T(0) : sl.c[g];
                }
            }
            b += G;
        };
        while (fl != uint64_t(1) << kSetBonds) {
            high(sa);
            add(sb);
            high(sb);
            add(sa);
        }
        if (set == 0 || n_high > set) {
#pragma unroll
            for (int i = 0; i < R; ++i) anti[i] = ah;
        }
        const int nb = n_bonds - set < kSetBonds ? n_bonds - set : kSetBonds;
        while (b < nb) {
            lows(sa);
            add(sb);
            lows(sb);
            add(sa);
        }
    }
    add(sb);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const uint32_t j = j0 + uint32_t(64 * i + lane);
        if constexpr (EPI == kEpiLanczos) {
#pragma unroll
            for (int c = 0; c < VB; ++c) prod[i][c] = 0.0;
        }
        if (j - jlo < jn) {
            const uint32_t t = run.base + j;
            T xt[VB], out[VB];
            load_row<T, VB>(reinterpret_cast<const T*>(xb + uint64_t(t) * ldb), xt);
            const T diag = jsum4 - anti[i];
#pragma unroll
            for (int c = 0; c < VB; ++c) out[c] = diag * xt[c] + acc[i][c];
            T* yrow = y + uint64_t(t - row0) * ld + col0;
            if constexpr (EPI == kEpiLanczos) {
                lanczos_epilogue<T, VB>(xt, out, yrow, ab, first, prod[i]);
            }
            store_row<T, VB>(yrow, out);
        }
    }
}

// y = H x on the sector rows [pos, end) by one wave, 64 R rows of a run at a
// time.
template <typename L, typename T, int VB, int R, int G>
__device__ __forceinline__ void run_rows(const SectorDev& S, const BondTable& B, const unsigned char* low, Binom C,
                                         int low_bits, const T* __restrict__ x, T* __restrict__ y, uint64_t ld,
                                         uint32_t col0, uint32_t row0, uint32_t pos, uint32_t end) {
    const int lane = threadIdx.x & 63;
    double none[R][VB];
    while (pos < end) {
        Run<L> run;
        run.find(pos, S, C, low_bits, lane);
        const uint32_t lim = end - run.base < run.size ? end : run.base + run.size;
        RunBonds<T> rb;
        rb.load(run, B, 0, low_bits, lane, reinterpret_cast<const unsigned char*>(x + col0), uint32_t(ld * sizeof(T)),
                S.dim - 1);
#pragma unroll 1
        for (; pos < lim; pos = lim - pos > uint32_t(64 * R) ? pos + uint32_t(64 * R) : lim)
            run_block<L, T, VB, R, G, kEpiPlain>(S, B, low, low_bits, run, rb, x, y, ld, col0, row0, pos, pos, lim,
                                                 nullptr, false, none);
    }
}

}  // namespace ftlm
