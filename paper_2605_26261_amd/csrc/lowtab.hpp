// Rank tables of the low part of a spin-1/2 label. The low kLowBits sites of
// a label take every pattern with a given number of up spins, in ascending
// order, under each pattern of the sites above them (a run of consecutive
// sector rows). The rank of a pattern among the patterns with its popcount
// does not depend on the sector, nor on how many of its leading bits are
// zero, so one table serves every sector and every low part of at most
// kLowBits sites.
#pragma once

#include <stdint.h>

namespace ftlm {

constexpr int kLowBits = 14;
constexpr int kLowSize = 1 << kLowBits;

struct LowTables {
    uint16_t rank[kLowSize];        // rank of l among the patterns with popcount(l) up spins
    uint16_t pattern[kLowSize];     // the patterns sorted by popcount, then by value
    uint32_t first[kLowBits + 2];   // where the patterns of a popcount begin
};

constexpr LowTables make_low_tables() {
    LowTables t{};
    uint32_t count[kLowBits + 1] = {};
    for (int l = 0; l < kLowSize; ++l) {
        const int k = __builtin_popcount(l);
        t.rank[l] = uint16_t(count[k]++);
    }
    for (int k = 0; k <= kLowBits; ++k) t.first[k + 1] = t.first[k] + count[k];
    for (int l = 0; l < kLowSize; ++l) {
        const int k = __builtin_popcount(l);
        t.pattern[t.first[k] + t.rank[l]] = uint16_t(l);
    }
    return t;
}

}  // namespace ftlm
