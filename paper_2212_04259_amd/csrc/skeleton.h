// Result of a skeleton search as held by the library (bns_skeleton handles).
#pragma once

#include <stdint.h>

#include <mutex>
#include <vector>

#include "../../include/bns.h"

// A search fills the compact form (removal depth per pair as int8, the
// sepsets of depth >= 1 in removal-record order), and the accessors answer
// from it: writing n x n arrays of the expanded form first cost a 1,000-
// variable search 2 ms of new pages.  Handles built on the host hold the
// arrays they were given (full = true).
struct bns_skeleton {
    int32_t n = 0;
    std::vector<int8_t> rdep;         // compact: n x n, removal depth or -1
    std::vector<int64_t> rec_pair;    // compact: i n + j (i < j) of each pool record
    std::vector<int64_t> rec_off;     // compact: its offset in pool
    std::vector<int32_t> pool;        // sepset members, ascending per pair
    std::vector<bns_depth_stats> stats;
    // full form
    std::vector<uint8_t> adj;     // n x n, 1 = edge kept
    std::vector<int32_t> depth;   // n x n, removal depth or -1
    std::vector<int64_t> sepoff;  // n x n, offset of the pair's sepset in pool or -1
    bool full = false;
    bool planes = false;  // a search that ran depths 0 and 1 from bit planes
    // compact: pool records by pair, made when a sepset is first asked for
    // (open addressing, record + 1, 0 = empty)
    mutable std::vector<uint32_t> slot;
    mutable std::once_flag once;

    int32_t depth_at(int64_t ij) const { return full ? depth[(size_t)ij] : (int32_t)rdep[(size_t)ij]; }
    bool kept(int64_t i, int64_t j) const {
        return i != j && (full ? adj[(size_t)(i * n + j)] != 0 : rdep[(size_t)(i * n + j)] < 0);
    }
    static size_t hash(int64_t pair) { return (size_t)(((uint64_t)pair * 0x9E3779B97F4A7C15ull) >> 20); }
    // Offset in pool of the sepset of a pair removed at depth >= 1.
    int64_t sepset_at(int64_t i, int64_t j) const {
        if (full) return sepoff[(size_t)(i * n + j)];
        std::call_once(once, [this] {
            size_t cap = 16;
            while (cap < 2 * rec_pair.size()) cap *= 2;
            slot.assign(cap, 0u);
            for (size_t r = 0; r < rec_pair.size(); ++r) {
                size_t h = hash(rec_pair[r]) & (cap - 1);
                while (slot[h]) h = (h + 1) & (cap - 1);
                slot[h] = (uint32_t)r + 1u;
            }
        });
        const int64_t pair = i < j ? i * n + j : j * n + i;
        const size_t mask = slot.size() - 1;
        for (size_t h = hash(pair) & mask; slot[h]; h = (h + 1) & mask)
            if (rec_pair[slot[h] - 1u] == pair) return rec_off[slot[h] - 1u];
        return -1;
    }
};
