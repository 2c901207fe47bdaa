// The library's host paths when memory is refused: run on the CPU against
// tests/fake_hip.cpp, one scenario per argument.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "fake_hip.h"
#include "tfmm.h"

#define CHECK(x)                                                                          \
    do {                                                                                  \
        if (!(x)) {                                                                       \
            std::printf("failed: %s (line %d, %s)\n", #x, __LINE__, fake.what.c_str());   \
            std::exit(1);                                                                 \
        }                                                                                 \
    } while (0)

static double arrays[64];  // stand for the caller's device arrays

struct Size {
    long n, leaves, levels;
};
static const Size kSizes[] = {{900, 30, 2}, {40000, 1500, 5}, {200000, 8000, 8}};

static void shape(const Size& s) {
    fake.leaves = s.leaves;
    fake.levels = s.levels;
    fake.near = 9 * s.leaves;
    fake.far = 40 * s.leaves;
}
static tfmm_ctx* make_ctx() {
    tfmm_ctx* c = nullptr;
    CHECK(tfmm_ctx_create(0, 0, &c) == TFMM_OK);
    return c;
}
static tfmm_tree* make_tree(tfmm_ctx* c, const Size& s) {
    shape(s);
    tfmm_tree* t = nullptr;
    int rc;
    while ((rc = tfmm_build_tree(c, s.n, arrays, arrays + 1, 64, nullptr, &t)) != TFMM_OK) CHECK(rc == TFMM_ENOMEM);
    return t;
}
static void drop(tfmm_tree* t, tfmm_ctx* c) {
    CHECK(tfmm_tree_destroy(t) == TFMM_OK);
    CHECK(tfmm_ctx_destroy(c) == TFMM_OK);
    CHECK(fake_all_gone());
}
// After a refused call nothing runs on the tree's own stream any more, which the
// caller's stream does not wait for.
static int evaluate(tfmm_tree* t, const tfmm_params& q, double* pot) {
    const int rc = tfmm_evaluate_forces(t, &q, arrays, pot, nullptr);
    if (rc != TFMM_OK)
        for (void* s : fake.busy) CHECK(s == nullptr);
    return rc;
}
// Evaluations of every kind; refused: how many may be for lack of memory.  What
// went well before a refused one goes well after it.
static void evaluations(tfmm_tree* t, int refused) {
    tfmm_params last{};
    for (int variant : {TFMM_STANDARD, TFMM_CONSERVING, TFMM_CONSERVING_R2})
        for (int p : {1, 2, 6, 4, 8, 5})
            for (int pot : {0, 1})
                for (int prec : {TFMM_MIXED32, TFMM_FP64, TFMM_MIXED32}) {
                    if (variant == TFMM_CONSERVING_R2 && p != 1) continue;
                    tfmm_params q{p, 0.5, 1e-3, 1.0, variant, prec, 0};
                    if (variant == TFMM_CONSERVING && p <= 5 && prec == TFMM_FP64) q.scalar_degree = p;
                    if (pot) q.theta = 0.6;
                    const int rc = evaluate(t, q, pot ? arrays + 1 : nullptr);
                    CHECK(rc == TFMM_OK || (rc == TFMM_ENOMEM && refused-- > 0));
                    if (rc == TFMM_OK) last = q;
                    else if (last.p) {
                        const int again = evaluate(t, last, nullptr);
                        CHECK(again == TFMM_OK || (again == TFMM_ENOMEM && refused-- > 0));
                    }
                }
}

// Every allocation refused in turn; the tree serves on as if nothing had been.
static void refused_memory() {
    for (const Size& s : kSizes)
        for (int overflow : {0, 1}) {
            long total = 0;
            for (long k = 0; k <= total; ++k) {
                tfmm_ctx* c = make_ctx();
                fake.what = "n " + std::to_string(s.n) + ", allocation " + std::to_string(k) + " refused";
                fake.overflow = overflow;
                fake.mallocs = 0;
                fake.fail_at = k;
                tfmm_tree* t = make_tree(c, s);
                evaluations(t, k ? 2 : 0);
                int rc;
                while ((rc = tfmm_tree_rebuild(t, s.n + 50, arrays, arrays + 1, nullptr)) != TFMM_OK)
                    CHECK(rc == TFMM_ENOMEM);
                evaluations(t, k ? 2 : 0);
                if (k == 0) total = fake.mallocs;
                fake.fail_at = 0;
                drop(t, c);
            }
            CHECK(total > 50);
        }
}

// A walk pass that gave up waiting for another workgroup leaves pairs unwritten:
// no list is made from them.
static void wait_ran_out() {
    for (const Size& s : kSizes)
        for (int walks : {1, 2}) {  // the first walk, and one sized by the walk before
            fake.what = "n " + std::to_string(s.n) + ", walk " + std::to_string(walks);
            tfmm_ctx* c = make_ctx();
            tfmm_tree* t = make_tree(c, s);
            if (walks == 2) CHECK(tfmm_tree_walk(t, 0.7, nullptr) == TFMM_OK);
            fake.list_launches = 0;
            fake.wait_ran_out = true;
            const tfmm_params q{4, 0.5, 1e-3, 1.0, TFMM_CONSERVING, TFMM_MIXED32, 0};
            CHECK(tfmm_evaluate_forces(t, &q, arrays, nullptr, nullptr) == TFMM_EDEVICE);
            CHECK(fake.list_launches == 0);
            fake.wait_ran_out = false;
            drop(t, c);
        }
}

// Pairs whose directed entries do not fit 32-bit offsets: refused before any list
// is made from them.
static void too_many_pairs() {
    for (int near : {0, 1})
        for (long pairs : {2147483648L, 4294967297L}) {
            fake.what = (near ? "near " : "far ") + std::to_string(pairs);
            tfmm_ctx* c = make_ctx();
            tfmm_tree* t = make_tree(c, kSizes[1]);
            (near ? fake.near : fake.far) = pairs;
            fake.list_launches = 0;
            const tfmm_params q{4, 0.5, 1e-3, 1.0, TFMM_CONSERVING, TFMM_MIXED32, 0};
            CHECK(tfmm_evaluate_forces(t, &q, arrays, nullptr, nullptr) == TFMM_ENOMEM);
            CHECK(fake.list_launches == 0);
            CHECK(tfmm_tree_walk(t, 0.5, nullptr) == TFMM_ENOMEM);
            shape(kSizes[1]);
            CHECK(tfmm_evaluate_forces(t, &q, arrays, nullptr, nullptr) == TFMM_OK);
            drop(t, c);
        }
}

// More partial sums than 32-bit offsets reach: refused before the near field.
static void too_many_rows() {
    for (const Size& s : kSizes)
        for (unsigned long long rows : {4294967295ull, 4294967296ull, 1ull << 40}) {
            fake.what = "n " + std::to_string(s.n) + ", rows " + std::to_string(rows);
            tfmm_ctx* c = make_ctx();
            tfmm_tree* t = make_tree(c, s);
            fake.rows = rows;
            fake.near_launches = 0;
            const tfmm_params q{4, 0.5, 1e-3, 1.0, TFMM_CONSERVING, TFMM_MIXED32, 0};
            const bool fits = rows <= 4294967295ull;
            CHECK(tfmm_evaluate_forces(t, &q, arrays, nullptr, nullptr) == (fits ? TFMM_OK : TFMM_ENOMEM));
            CHECK((fake.near_launches > 0) == fits);
            fake.rows = 0;
            CHECK(tfmm_evaluate_forces(t, &q, arrays, nullptr, nullptr) == TFMM_OK);
            drop(t, c);
        }
}

// What fits with a walk that takes its room as it goes is not refused for the
// larger room that is estimated for a first walk.
static void first_walk_memory() {
    for (const Size& s : {kSizes[1], kSizes[2]}) {
        tfmm_params q{8, 0.5, 1e-3, 1.0, TFMM_CONSERVING, TFMM_FP64, 0};
        // the bytes of a solve with the estimate, and of one without
        auto solve = [&](size_t budget, size_t limit, bool must) {
            fake.what = "n " + std::to_string(s.n) + ", p " + std::to_string(q.p) + ", budget " +
                        std::to_string(budget) + ", device " + std::to_string(limit);
            tfmm_ctx* c = make_ctx();
            CHECK(tfmm_ctx_set_budget(c, budget) == TFMM_OK);
            fake.limit = limit;
            fake.sized_passes = 0;
            shape(s);
            tfmm_tree* t = nullptr;
            int rc = tfmm_build_tree(c, s.n, arrays, arrays + 1, 64, nullptr, &t);
            if (rc == TFMM_OK) rc = evaluate(t, q, nullptr);
            CHECK(rc == TFMM_OK || (rc == TFMM_ENOMEM && !must));
            const size_t held = rc == TFMM_OK ? tfmm_ctx_bytes_in_use(c) : 0;
            fake.limit = 0;
            drop(t, c);
            return held;
        };
        for (int p : {2, 6, 8}) {
            q.p = p;
            const size_t estimated = solve(0, 0, true);
            CHECK(fake.sized_passes == 0);
            size_t sized = 0;  // the least that a budget admits
            for (size_t b = estimated / 8; !sized; b += b / 50) sized = solve(b, 0, false) ? b : 0;
            CHECK(sized < estimated && (p > 2 || fake.sized_passes > 0));
            for (size_t b = sized; b < 3 * estimated; b += b / 25) solve(b, 0, true);
            for (size_t d = sized + sized / 50; d < 2 * estimated; d += d / 25) solve(0, d, true);
        }
        // a second tree finds what the first one's estimate left over
        fake.what = "two trees";
        const size_t sized = [&] {
            for (size_t b = 1 << 20;; b += b / 50)
                if (solve(b, 0, false)) return b;
        }();
        tfmm_ctx* c = make_ctx();
        CHECK(tfmm_ctx_set_budget(c, 4 * sized) == TFMM_OK);
        std::vector<tfmm_tree*> trees;
        for (int k = 0; k < 3; ++k) {
            trees.push_back(nullptr);
            CHECK(tfmm_build_tree(c, s.n, arrays, arrays + 1, 64, nullptr, &trees.back()) == TFMM_OK);
            CHECK(evaluate(trees.back(), q, nullptr) == TFMM_OK);
        }
        for (tfmm_tree* t : trees) CHECK(tfmm_tree_destroy(t) == TFMM_OK);
        CHECK(tfmm_ctx_destroy(c) == TFMM_OK);
        // a walked tree that needs more later, on a device that is full by then
        fake.what = "later";
        c = make_ctx();
        tfmm_tree* t = make_tree(c, s);
        q.p = 1;
        CHECK(evaluate(t, q, nullptr) == TFMM_OK);
        CHECK(tfmm_ctx_trim(c) == TFMM_OK);
        fake.limit = fake.bytes;
        q.p = 3;
        CHECK(evaluate(t, q, nullptr) == TFMM_OK);
        int64_t info[8];
        CHECK(tfmm_tree_info(t, info) == TFMM_OK && info[4] == fake.far && info[5] == fake.near);
        CHECK(tfmm_tree_rebuild(t, s.n + s.n / 10, arrays, arrays + 1, nullptr) == TFMM_OK);
        fake.limit = 0;
        drop(t, c);
    }
}

// A walk's passes by their size: one launch up to 2^24 entries, two beyond, and
// neither waits for the host.
static void pass_sizes() {
    for (long entries : {2000L, 13421721L, 13421725L, 40000000L}) {  // a quarter more is expected
        fake.what = std::to_string(entries) + " entries";
        tfmm_ctx* c = make_ctx();
        tfmm_tree* t = make_tree(c, kSizes[1]);
        fake.pass_entries = entries;
        CHECK(tfmm_tree_walk(t, 0.5, nullptr) == TFMM_OK);
        fake.pass_launches = fake.emit_launches = fake.sized_passes = 0;
        CHECK(tfmm_tree_walk(t, 0.6, nullptr) == TFMM_OK);
        const bool one = entries + entries / 4 + 64 <= 1L << 24;
        CHECK(fake.pass_launches == (one ? 1 : 0) && fake.emit_launches == (one ? 0 : 1) && fake.sized_passes == 0);
        fake.pass_entries = 3000;
        drop(t, c);
    }
}

int main(int, char** argv) {
    for (const double& x : arrays) fake.user.insert(&x);
    const std::string what = argv[1];
    if (what == "refused_memory") refused_memory();
    else if (what == "wait_ran_out") wait_ran_out();
    else if (what == "too_many_pairs") too_many_pairs();
    else if (what == "too_many_rows") too_many_rows();
    else if (what == "first_walk_memory") first_walk_memory();
    else if (what == "pass_sizes") pass_sizes();
    else return 2;
    std::puts("host paths ok");
    return 0;
}
