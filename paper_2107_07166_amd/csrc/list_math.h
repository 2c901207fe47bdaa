// Arithmetic of the near-field work items, free of HIP so that a test can run it
// on the CPU too.
#pragma once

#include <cstdint>

namespace tfmm {

// The workgroups of a walk pass in one launch, at most kPassGrid, hand their output
// counts on in words of kCountBits bits per kind.  A workgroup takes up to nf /
// kPassGrid + 8 of the pass's nf entries, and an entry gives at most 15 outputs of a
// kind (seven pairs of its run split, and one self pair with eight children), so
// the counts of up to kPassMax entries fit whatever becomes of them.  Larger passes
// run in two launches.
constexpr int kPassGrid = 256;
constexpr int kCountBits = 20;
constexpr int64_t kPassMax = (int64_t)kPassGrid << (kCountBits - 4);

// List offsets and entry counts have 32 bits, and loops over the entries step past
// the last one by less than kListStep: the most pairs whose directed entries (two
// each) leave room for that.
constexpr uint32_t kListStep = 1u << 20;
constexpr int64_t kMaxPairs = (((int64_t)1 << 32) - kListStep) / 2;
constexpr bool lists_fit(int64_t far_pairs, int64_t near_pairs) {
    return far_pairs <= kMaxPairs && near_pairs <= kMaxPairs;
}

// A target leaf's near list is cut before entry q when the number of source
// particles preceding q in that list crosses a multiple of kItemSources, so no
// wavefront receives more than about kItemSources sources per target.
constexpr uint32_t kItemSources = 4096;

// What a source leaf adds to the prefixes P that the lists are cut by: its
// particles, and kItemSources if it holds more, as a leaf of the deepest level
// may whose particles (nearly) coincide.  With no more than that per entry the
// item index grows by at most one from an entry to the next: every item has a
// first entry of its own, and a list has no more items than entries.
constexpr uint32_t source_step(int32_t count) {
    return (uint32_t)count < kItemSources ? (uint32_t)count : kItemSources;
}

// Items of the list of entries [q0, q1): entry q belongs to item
// floor((P[q] - P[q0]) / kItemSources).  P is taken modulo 2^32; only differences
// inside one list are used.
constexpr uint32_t list_items(const uint32_t* P, uint32_t q0, uint32_t q1) {
    return q1 > q0 ? (P[q1 - 1u] - P[q0]) / kItemSources + 1u : 0u;
}

// Partial-sum rows of a list of n items (one per item and target particle): only a
// leaf split into several items needs any.  Offsets into them have 32 bits; the
// total is kept in 64 to see whether they do.
constexpr uint64_t item_rows(uint32_t n, int32_t targets) { return n > 1u ? (uint64_t)n * (uint32_t)targets : 0u; }
constexpr bool rows_fit(uint64_t rows) { return rows <= 0xffffffffull; }

// First entry of item k of the list: the first q with P[q] - P[q0] >= k
// kItemSources, by binary search.
constexpr uint32_t item_start(const uint32_t* P, uint32_t q0, uint32_t q1, uint32_t k) {
    if (k == 0u) return q0;
    const uint32_t p0 = P[q0], want = k * kItemSources;
    uint32_t lo = q0 + 1u, hi = q1 - 1u;
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2u;
        if (P[mid] - p0 >= want) hi = mid;
        else lo = mid + 1u;
    }
    return lo;
}

}  // namespace tfmm
