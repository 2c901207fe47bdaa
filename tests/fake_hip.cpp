#include "fake_hip.h"

#include <cxxabi.h>

#include <cstdio>
#include <cstdlib>
#include <map>
#include <utility>
#include <vector>

#include "common.h"

using namespace tfmm;

FakeHip fake;

namespace {

using Kernel = std::pair<std::string, std::vector<std::string>>;  // name, parameter types
std::map<const void*, Kernel>& kernels() {
    static auto* m = new std::map<const void*, Kernel>;
    return *m;
}
std::map<char*, size_t> device, pinned;
std::set<void*> streams, events;
std::map<const void*, int> moments;  // order of the moments in an allocation

[[noreturn]] void die(const std::string& m) {
    std::printf("fake HIP: %s (%s)\n", m.c_str(), fake.what.c_str());
    std::fflush(stdout);
    std::abort();
}
bool within(const std::map<char*, size_t>& m, const void* p) {
    auto it = m.upper_bound((char*)p);
    if (it == m.begin()) return false;
    --it;
    return (char*)p <= it->first + it->second;
}
bool live(const void* p) { return within(device, p) || within(pinned, p) || fake.user.count(p); }
void check(hipStream_t s) {
    if (s && !streams.count(s)) die("dead stream");
}
void check(hipEvent_t e) {
    if (!events.count(e)) die("dead event");
}
bool has(const std::string& n, const char* s) { return n.find(s) != std::string::npos; }
int order_of(const std::string& n) { return std::atoi(n.c_str() + n.find('<') + 1); }

// Pointers that may be null: the optional inputs and outputs.
bool null_ok(const std::string& n, size_t k) {
    if (has(n, "p2p_reduce")) return k >= 8;
    if (has(n, "p2p_")) return k >= 13;  // the potential's
    return has(n, "bucket_") || has(n, "bbox") || has(n, "morton") || has(n, "gather") || has(n, "leaf_level") ||
           has(n, "radix_pass") || has(n, "diag_pass") || has(n, "csr_offsets");
}

// The read-backs' layouts.
struct Header {
    int64_t LB[kLevels + 2], max_level, n_nodes, n_leaves, nonfinite;
};
struct Slot {
    uint32_t nf, buf;
    unsigned long long n_far, n_near;
};
struct State {
    Slot slot[2];
    uint32_t overflow, passes, max_nf, pad, nf_pass[64];
};
struct Totals {
    uint32_t multi, near_entries, items, partial;
    unsigned long long rows;
};
bool sized_pass = false;  // a host-sized walk pass waits for its totals
void post(const Mailbox& m, const void* src, size_t bytes) {
    std::memcpy(m.box + kBoxHeaderWords, src, bytes);
    m.box[1] = *m.err;
    m.box[0] = m.seq;
}

void answer(const std::string& n, void** a) {
    if (has(n, "slot_scan_kernel")) {
        // a tower: the roots, levels of eight nodes, one level of leaves
        Header h{};
        int64_t at = *(int*)a[5];
        for (int k = 1; k <= kLevels + 1; ++k) {
            h.LB[k] = at;
            at += k < fake.levels ? 8 : (k == fake.levels ? fake.leaves : 0);
        }
        h.max_level = fake.levels;
        h.n_nodes = h.LB[kLevels + 1];
        h.n_leaves = fake.leaves;
        h.nonfinite = fake.nonfinite;
        std::memcpy(*(void**)a[6], &h, sizeof h);
        post(*(Mailbox*)a[7], &h, sizeof h);
    } else if (has(n, "walk_seq_kernel")) {
        const Mailbox m = *(Mailbox*)a[9];
        const int slot = *(int*)a[3];
        State s{};
        s.slot[slot ^ 1] = {0, 0, (unsigned long long)fake.far, (unsigned long long)fake.near};
        s.passes = 5;
        s.max_nf = (uint32_t)fake.pass_entries;
        for (int k = 0; k < 5; ++k) s.nf_pass[k] = k == 2 ? s.max_nf : 100;
        s.overflow = fake.overflow > 0;
        std::memcpy(*(void**)a[2], &s, sizeof s);
        if (m.box) {
            if (fake.wait_ran_out) *const_cast<uint32_t*>(m.err) = 1u;
            if (fake.overflow > 0) --fake.overflow;
            post(m, &s, sizeof s);
        }
    } else if (has(n, "items_small_kernel")) {
        const Totals t{0u, (uint32_t)(2 * fake.near - fake.leaves), (uint32_t)fake.leaves, 0u, fake.rows};
        post(*(Mailbox*)a[15], &t, sizeof t);
    } else if (has(n, "walk_pass_kernel")) {
        ++fake.pass_launches;
    } else if (has(n, "walk_emit_kernel")) {
        ++fake.emit_launches;
    } else if (has(n, "walk_total_kernel")) {
        ++fake.sized_passes;
        sized_pass = true;
    } else if (has(n, "mailbox_kernel")) {
        const int nw = *(int*)a[2];
        std::vector<uint32_t> v((size_t)nw, 0u);
        if (sized_pass) {  // the first one gives every pair
            const unsigned long long t[3] = {0ull, (unsigned long long)fake.far, (unsigned long long)fake.near};
            std::memcpy(v.data(), t, sizeof t);
            sized_pass = false;
        } else if (nw == (int)sizeof(Totals) / 4) {
            const Totals t{1u, (uint32_t)(2 * fake.near - fake.leaves), (uint32_t)fake.leaves + 3u, 100u, fake.rows};
            std::memcpy(v.data(), &t, sizeof t);
        }
        post(*(Mailbox*)a[0], v.data(), (size_t)nw * 4);
    } else if (has(n, "p2m_kernel")) {
        moments[*(void**)a[6]] = moments[*(void**)a[7]] = order_of(n);
    } else if (has(n, "m2l_")) {
        const void* W = *(void**)a[4];
        if (!moments.count(W)) die("M2L reads memory without moments: " + n);
        if (has(n, "m2l_kernel") && *(int64_t*)a[5] != round_up(c_le(moments[W]), 4)) die("M2L with moments of order " + std::to_string(moments[W]));
        if (has(n, "cons_pass") && moments[W] != order_of(n)) die("M2L with moments of order " + std::to_string(moments[W]));
    }
    if (has(n, "p2p_")) ++fake.near_launches;
    if (has(n, "bucket_") || has(n, "radix_hist") || has(n, "p2p_")) ++fake.list_launches;
}

}  // namespace

bool fake_all_gone() { return device.empty() && pinned.empty() && streams.empty() && events.empty(); }

extern "C" {

struct Config {
    dim3 g, b;
    size_t shared;
    hipStream_t s;
};
static std::vector<Config> configs;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shared, hipStream_t s) {
    configs.push_back({g, b, shared, s});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shared, hipStream_t* s) {
    const Config c = configs.back();
    configs.pop_back();
    *g = c.g;
    *b = c.b;
    *shared = c.shared;
    *s = c.s;
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* stub, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
    int status;
    char* d = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    const std::string s = d ? d : name;
    std::free(d);
    // the parameters: the last top-level parentheses
    const size_t e = s.rfind(')');
    size_t i = e;
    for (int depth = 0;; --i) {
        if (s[i] == ')') ++depth;
        if (s[i] == '(' && --depth == 0) break;
    }
    std::vector<std::string> par(1);
    int depth = 0;
    for (size_t k = i + 1; k < e; ++k) {
        const char c = s[k];
        if (c == '<' || c == '(') ++depth;
        if (c == '>' || c == ')') --depth;
        if (c == ',' && depth == 0) par.emplace_back();
        else par.back() += c;
    }
    kernels()[stub] = {s.substr(0, i), par};
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, hipStream_t s) {
    const auto it = kernels().find(f);
    if (it == kernels().end()) die("unknown kernel");
    const auto& [name, par] = it->second;
    check(s);
    if (g.x == 0 || g.y == 0 || b.x == 0 || b.x > 1024) die("launch shape of " + name);
    for (size_t k = 0; k < par.size(); ++k) {
        if (par[k].empty() || par[k].back() != '*') continue;
        const void* p = *(void**)args[k];
        if (p ? !live(p) : !null_ok(name, k))
            die("argument " + std::to_string(k) + " (" + par[k] + ") of " + name + (p ? " is not live" : " is null"));
    }
    ++fake.launches;
    fake.busy.insert(s);
    answer(name, args);
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
    ++fake.mallocs;
    if (fake.limit && fake.bytes + n > fake.limit) return hipErrorOutOfMemory;
    if (fake.fail_at && (fake.mallocs == fake.fail_at || fake.mallocs == fake.fail_at + 1)) {
        if (fake.mallocs > fake.fail_at) fake.fail_at = 0;
        return hipErrorOutOfMemory;
    }
    *p = std::malloc(n);
    device[(char*)*p] = n;
    fake.bytes += n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (!p) return hipSuccess;
    const auto it = device.find((char*)p);
    if (it == device.end()) die("hipFree of dead memory");
    fake.bytes -= it->second;
    device.erase(it);
    moments.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::malloc(n);
    pinned[(char*)*p] = n;
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    if (!pinned.erase((char*)p)) die("hipHostFree of dead memory");
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
    *d = h;
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
    check(st);
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) {
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "fake HIP error"; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
    static double scratch[1 << 14];
    fake.user.insert(scratch);
    *p = scratch;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
    fake.busy.clear();
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = (hipStream_t)std::malloc(8);
    streams.insert(*s);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    if (!streams.erase(s)) die("dead stream destroyed");
    fake.busy.erase(s);
    std::free(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    check(s);
    fake.busy.erase(s);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    check(s);
    check(e);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = (hipEvent_t)std::malloc(8);
    events.insert(*e);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
    if (!events.erase(e)) die("dead event destroyed");
    std::free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    check(e);
    check(s);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    check(e);
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
    check(a);
    check(b);
    *ms = 1.f;
    return hipSuccess;
}

}  // extern "C"
