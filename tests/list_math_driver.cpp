// Host checks of csrc/list_math.h (built with the address and undefined-behaviour
// sanitizers): the near-field work items of lists whose source leaves hold up to
// a million particles.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "list_math.h"

using namespace tfmm;

#define CHECK(x)                                                        \
    do {                                                                \
        if (!(x)) {                                                     \
            std::printf("failed: %s (line %d)\n", #x, __LINE__);        \
            return 1;                                                   \
        }                                                               \
    } while (0)

// One list of the given source counts, its prefixes starting at base.
static int check_list(const std::vector<int32_t>& count, uint32_t base) {
    const uint32_t q0 = 3u, q1 = q0 + (uint32_t)count.size();
    std::vector<uint32_t> P(q1);
    uint32_t run = base;
    for (uint32_t q = q0; q < q1; ++q) {
        P[q] = run;
        run += source_step(count[q - q0]);
    }
    const uint32_t n = list_items(P.data(), q0, q1);
    CHECK(n <= q1 - q0);
    CHECK((n == 0u) == (q1 == q0));
    uint32_t at = q0;
    for (uint32_t k = 0; k < n; ++k) {
        const uint32_t a = item_start(P.data(), q0, q1, k);
        const uint32_t b = k + 1u < n ? item_start(P.data(), q0, q1, k + 1u) : q1;
        CHECK(a == at && b > a);  // consecutive and not empty
        uint64_t sources = 0;
        for (uint32_t q = a; q < b; ++q) sources += source_step(count[q - q0]);
        CHECK(sources < 2u * kItemSources);
        at = b;
    }
    CHECK(at == q1 || n == 0u);
    return 0;
}

int main() {
    // as many particles as an ordinary leaf may hold: the count itself
    CHECK(source_step(1) == 1u && source_step(4095) == 4095u && source_step(4096) == 4096u);
    CHECK(source_step(4097) == 4096u && source_step(1 << 30) == 4096u);
    // the counts of the largest pass in one launch, with every workgroup's share at its worst
    CHECK(15 * (kPassMax / kPassGrid + 8) < (int64_t)1 << kCountBits && 3 * kCountBits <= 62);
    // the directed entries of the most pairs, and a loop's last step past them
    CHECK(lists_fit(0, 0) && lists_fit(kMaxPairs, kMaxPairs));
    CHECK(!lists_fit(kMaxPairs + 1, 0) && !lists_fit(0, kMaxPairs + 1) && !lists_fit((int64_t)1 << 31, 0));
    CHECK(2ull * kMaxPairs + (kListStep - 1u) <= 0xffffffffull);
    CHECK(item_rows(0, 64) == 0 && item_rows(1, 64) == 0 && item_rows(3, 64) == 192);
    CHECK(item_rows(1u << 20, 1 << 30) == 1ull << 50);
    CHECK(rows_fit(0) && rows_fit(4294967295ull) && !rows_fit(4294967296ull) && !rows_fit(1ull << 50));
    std::mt19937 rng(1);
    std::vector<std::vector<int32_t>> lists = {{}, {1}, {4096}, {1000000}, {1, 1000000, 1}, {1000000, 1000000},
                                               {4, 4, 4, 1000000, 4, 4, 4}, std::vector<int32_t>(5000, 5000)};
    for (int k = 0; k < 200; ++k) {
        std::vector<int32_t> c(rng() % 300);
        for (auto& x : c) x = 1 + (int32_t)(rng() % 20 == 0 ? rng() % 1000000 : rng() % 64);
        lists.push_back(c);
    }
    for (const auto& c : lists)
        for (uint32_t base : {0u, 4095u, 0xfffff000u})  // the prefixes wrap
            if (check_list(c, base)) return 1;
    std::puts("list math ok");
    return 0;
}
