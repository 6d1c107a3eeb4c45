// Tables of the low part of a general-spin label (digits 0 .. d - 1). Under
// each pattern of the sites above them the low sites take every digit string
// with the remaining digit sum, in ascending order (a run of consecutive sector
// rows). The rank of a string among those with its digit sum does not depend
// on the sector, so one table per d serves every one.
#pragma once

#include <stdint.h>

namespace ftlm {

// Low sites for 3 <= d <= 6: as many as leave a table of at most 8192 strings
// (16 KB of ranks in LDS).
constexpr int spin_low_sites(int d) { return d == 3 ? 8 : d == 4 ? 6 : 5; }

template <int D>
struct SpinLowTable {
    static constexpr int sites = spin_low_sites(D);
    static constexpr int size() {
        int n = 1;
        for (int i = 0; i < sites; ++i) n *= D;
        return n;
    }
    uint16_t rank[size()];               // rank of string l among those with its digit sum
    uint32_t digits[size()];             // the strings sorted by digit sum, then by value: four bits a site
    uint32_t first[sites * (D - 1) + 2];  // where the strings of a digit sum begin
};

template <int D>
constexpr SpinLowTable<D> make_spin_low_table() {
    SpinLowTable<D> t{};
    constexpr int n = SpinLowTable<D>::size(), sums = SpinLowTable<D>::sites * (D - 1) + 1;
    uint16_t sum[n] = {};
    uint32_t dig[n] = {};
    uint32_t count[sums] = {};
    for (int l = 0; l < n; ++l) {
        sum[l] = uint16_t(l == 0 ? 0 : sum[l / D] + l % D);
        dig[l] = l == 0 ? 0u : (dig[l / D] << 4) | uint32_t(l % D);
        t.rank[l] = uint16_t(count[sum[l]]++);
    }
    for (int k = 0; k < sums; ++k) t.first[k + 1] = t.first[k] + count[k];
    for (int l = 0; l < n; ++l) t.digits[t.first[sum[l]] + t.rank[l]] = dig[l];
    return t;
}

}  // namespace ftlm
