// Mutual dual-tree walk (the per-target interaction lists: lists.hip).
//
// The walk decides unordered node pairs level-synchronously from (root, root)
// (one such pair per set of a forest; the children of a pair belong to its
// set, so nodes of different sets never meet, and each set may have its own
// theta).  For each pair:
//   A == B : a leaf gives a near (P2P) self pair; otherwise the children
//            pairs (c_i, c_j), i <= j, are decided in the next pass;
//   A != B : R = sqrt((dx*dx + dy*dy) + dz*dz), d = Z_A - Z_B.  The pair is a
//            far (M2L) pair iff R > 0 and r_A + r_B <= theta * R
//            (Eq. mac_criterion with theta = tan of the MAC angle); else two
//            leaves give a near pair; else one node is split (the non-leaf
//            if one is a leaf, else the larger r_max, then the lower level,
//            then the lower index) and its children are paired with the other.
// A pass's frontier holds runs of sibling pairs: entry (f, O) stands for the
// pairs of O with node f and every later sibling of f.  A split gives one
// entry, a self pair one per child c_i (the run from c_i against c_i).
// Eight lanes take an entry, one pair each, so sibling records are read
// together and only the split pairs, about one in six, are written and read
// back.  Counts are compacted with prefix sums, so the emitted lists are in a
// fixed order (the frontier's, pass after pass) and the pair sets do not
// depend on scheduling.  FP64 without contraction so that every decision is
// reproducible.
#pragma clang fp contract(off)

#include <algorithm>
#include <cmath>

#include "common.h"
#include "list_math.h"

namespace tfmm {
namespace {

constexpr int TB = 256;

// Per node, packed for the walk by the tree build: geo = (centre of mass x, y, z, r_max),
// top = (child count + 16 x the siblings from this node to its last, level,
// first child, set).  theta: per set (forests walked with several thetas),
// else nullptr and the passes' scalar applies.
struct WalkNodes {
    const double4* __restrict__ geo;
    const int4* __restrict__ top;
    const double* theta;
    int32_t nn;
};

constexpr int kRun = 8;  // lanes per frontier entry: the most siblings

// The records of the pair of this lane, node A = f + x of entry (f, O) with x =
// lane % kRun.  All five are read at once, also where the run is shorter than x
// (the node index is kept in range) or the pair is a self pair: the passes are
// bound by the latency of these reads, and with the tests in between they were
// four round trips instead of one.
struct PairRecords {
    int32_t A, O;
    int sib;  // nodes in the run (0 past the frontier's end)
    int4 ta, to;
    double4 ga, go;
};

__device__ __forceinline__ PairRecords load_pair(const WalkNodes& w, bool valid, int2 e, int x) {
    PairRecords r;
    const int32_t last = w.nn - 1;
    r.A = e.x + x;
    r.O = e.y;
    const int32_t A = r.A < last ? r.A : last;
    const int sib = w.top[e.x].x >> 4;
    r.ta = w.top[A];
    r.to = w.top[r.O];
    r.ga = w.geo[A];
    r.go = w.geo[r.O];
    r.sib = valid ? sib : 0;
    return r;
}

// What becomes of a pair: bits 0-1 kind (0 near, 1 far, 2 expand self, 3
// split), bit 2 set when the split node is O; -1 where there is no pair.
__device__ __forceinline__ int decide(const WalkNodes& w, const PairRecords& r, int x, double theta) {
    if (x >= r.sib) return -1;
    const int na = r.ta.x & 15, no = r.to.x & 15;
    if (r.A == r.O) return na == 0 ? 0 : 2;
    const double dx = r.ga.x - r.go.x, dy = r.ga.y - r.go.y, dz = r.ga.z - r.go.z;
    const double R = sqrt((dx * dx + dy * dy) + dz * dz);
    const double ra = r.ga.w, ro = r.go.w;
    const double th = w.theta ? w.theta[r.ta.w] : theta;
    if (R > 0.0 && ra + ro <= th * R) return 1;
    if (na == 0 && no == 0) return 0;
    bool second;
    if (na == 0) second = true;
    else if (no == 0) second = false;
    else if (ra != ro) second = ro > ra;
    else if (r.ta.y != r.to.y) second = r.to.y < r.ta.y;
    else second = r.O < r.A;
    return second ? 7 : 3;
}

__device__ __forceinline__ uint64_t lanes_below() {
    const int lane = threadIdx.x & (kWave - 1);
    return lane == 0 ? 0ull : (~0ull >> (kWave - lane));
}

// Entries that a self pair adds: one per child.  Summed over the wavefront
// (self pairs are rare), and over the lanes below this one.
__device__ __forceinline__ uint32_t self_entries(int code, int nc, uint32_t& below) {
    const int lane = threadIdx.x & (kWave - 1);
    uint64_t m = __ballot(code == 2);
    below = 0u;
    uint32_t tot = 0u;
    while (m) {
        const int l = __ffsll((long long)m) - 1;
        const uint32_t c = (uint32_t)__builtin_amdgcn_readlane(nc, l);
        if (l < lane) below += c;
        tot += c;
        m &= m - 1ull;
    }
    return tot;
}

struct U3 {
    uint32_t a, b, c;  // next-frontier entries, far pairs, near pairs
};
__device__ __forceinline__ U3 u3add(U3 x, U3 y) { return {x.a + y.a, x.b + y.b, x.c + y.c}; }

// Outputs of the wavefront's pairs and of the lanes below this one (nc: the
// child count of the lane's split node).
__device__ __forceinline__ U3 wave_counts(int code, int nc, U3& below) {
    const uint64_t lt = lanes_below();
    const uint64_t mn = __ballot(code == 0), mf = __ballot(code == 1), ms = __ballot((code & 3) == 3 && code >= 0);
    const uint32_t self = self_entries(code, nc, below.a);
    below.a += (uint32_t)__popcll(ms & lt);
    below.b = (uint32_t)__popcll(mf & lt);
    below.c = (uint32_t)__popcll(mn & lt);
    return {(uint32_t)__popcll(ms) + self, (uint32_t)__popcll(mf), (uint32_t)__popcll(mn)};
}

// Writes the lane's output at its place (ts: the record of its split node);
// sink(i, entry) takes a next-frontier entry.
template <typename Sink>
__device__ __forceinline__ void lane_emit(int code, int32_t A, int32_t O, const int4& ts, unsigned long long on,
                                          unsigned long long ofar, unsigned long long onear, int2* __restrict__ far,
                                          int2* __restrict__ near, Sink sink) {
    const int2 pr = make_int2(A < O ? A : O, A < O ? O : A);
    if (code == 0) {
        near[onear] = pr;
    } else if (code == 1) {
        far[ofar] = pr;
    } else if (code >= 0) {
        if (code == 2) {
            for (int c = 0; c < (ts.x & 15); ++c) sink(on + c, make_int2(ts.z + c, ts.z + c));
        } else {
            sink(on, make_int2(ts.z, code == 7 ? A : O));
        }
    }
}

// Pass totals are carried in 64 bits so that a pass too large for 32-bit
// offsets is detected instead of wrapping.
struct U3L {
    unsigned long long a, b, c;
};
__device__ __forceinline__ U3L u3ladd(U3L x, U3 y) { return {x.a + y.a, x.b + y.b, x.c + y.c}; }
__device__ __forceinline__ U3L u3ladd(U3L x, U3L y) { return {x.a + y.a, x.b + y.b, x.c + y.c}; }

// Sum over the block (every thread calls it and gets the total).
__device__ __forceinline__ U3L block_sum(U3L x, U3L* wsum) {
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        x.a += __shfl_xor(x.a, d, kWave);
        x.b += __shfl_xor(x.b, d, kWave);
        x.c += __shfl_xor(x.c, d, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) wsum[threadIdx.x / kWave] = x;
    __syncthreads();
    U3L t{0ull, 0ull, 0ull};
#pragma unroll
    for (int k = 0; k < TB / kWave; ++k) t = u3ladd(t, wsum[k]);
    __syncthreads();
    return t;
}

// ---- frontier passes ----------------------------------------------------------
// The frontier's size and the running list lengths live on the device in two
// slots (a launch reads one and writes the other), so launches can be queued
// without reading anything back.  A pass whose outputs would not fit sets a
// sticky flag and writes nothing; later passes then see an empty frontier.
constexpr int kMaxPasses = 64;  // a walk needs at most 2 * 21 + 1 passes
struct WalkSlot {
    uint32_t nf, buf;  // frontier entries, and the buffer (0, 1) that holds them
    unsigned long long n_far, n_near;
};
struct WalkState {
    WalkSlot slot[2];
    uint32_t overflow;
    uint32_t passes;  // passes run
    uint32_t max_nf;  // largest frontier seen
    uint32_t pad;
    uint32_t nf_pass[kMaxPasses];  // frontier size of every pass (sizes the next walk's launches)
};
struct WalkOut {
    int2* fr[2];  // frontier buffers
    int2 *far, *near;
    unsigned long long cap_next, cap_far, cap_near;
};
constexpr int kWalkGrid = 1024;

// What the workgroups of a pass tell each other, per slot (a pass uses its own
// and clears the other's): start tickets, and the output counts of every
// workgroup in one word (kCountBits each of next, far and near; bit 63 set, bit 62
// if a count does not fit).
struct PassSync {
    unsigned long long counts[2][kPassGrid];
    uint32_t ticket[2];
};

// Whether a pass's totals T fit.
__device__ __forceinline__ bool pass_fits(const WalkOut& o, const U3L& T, const WalkSlot& s) {
    const unsigned long long lim = 0xffffffffull;
    return T.a <= o.cap_next && T.b <= lim && T.c <= lim && s.n_far + T.b <= o.cap_far && s.n_near + T.c <= o.cap_near;
}

__device__ __forceinline__ void pass_done(WalkState* st, WalkSlot* out, const WalkSlot& s, const U3L& T) {
    *out = WalkSlot{(uint32_t)T.a, s.buf ^ 1u, s.n_far + T.b, s.n_near + T.c};
    if (st->passes < (uint32_t)kMaxPasses) st->nf_pass[st->passes] = s.nf;
    st->passes += 1u;
    if ((uint32_t)T.a > st->max_nf) st->max_nf = (uint32_t)T.a;
}

// Small passes, one after another, in a single workgroup: a pass of up to
// limit entries is decided (the decisions kept in LDS), its counts scanned over
// the wavefronts, and its outputs written, with two barriers and no launch in
// between.  The frontier stays in LDS (and is written to memory too, for the
// launch that takes over).  With init, starts from the pairs (k, k) of the
// roots.  Stops when the frontier is empty or larger than limit.  A pass here
// takes 5 to 9 us (latency: one workgroup cannot hide it), a launch of its own
// 6 to 9 and the gap before it.  A small tree's walk is this one
// launch: Plummer 10007, built and solved in one call, 1070 -> 711 us together
// with the estimated room of a first walk.
constexpr int SQ = 1024;          // threads
constexpr int kSeqMax = 2048;     // most entries of a pass run here
constexpr int kSeqHead = 1024;    // a walk whose passes stay below this is run here whole
// The first and last passes of a walk with larger ones (100000 particles 734 us
// with 1024, 719 with 256; 20011 in FP64 557 and 552).
constexpr int kSeqEnds = 256;
__global__ __launch_bounds__(SQ) void walk_seq_kernel(WalkNodes w, WalkOut o, WalkState* __restrict__ st, int slot,
                                                      int init, int n_roots, uint32_t limit, double theta,
                                                      PassSync* __restrict__ sync, Mailbox mb) {
    constexpr int NW = SQ / kWave;
    constexpr int EPW = kWave / kRun;  // entries per wavefront and step
    __shared__ int2 fr[2][kSeqMax];
    __shared__ int8_t dec[kSeqMax * kRun];
    __shared__ U3 wtot[NW];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave, x = lane % kRun;
    for (int k = tid; k < kPassGrid; k += SQ) sync->counts[0][k] = sync->counts[1][k] = 0ull;
    if (tid < 2) sync->ticket[tid] = 0u;
    WalkSlot s;
    if (init) {
        s = WalkSlot{(uint32_t)n_roots, 0u, 0ull, 0ull};
        for (int k = tid; k < n_roots; k += SQ) {
            o.fr[0][k] = make_int2(k, k);
            if (k < kSeqMax) fr[0][k] = make_int2(k, k);
        }
        if (tid < kMaxPasses) st->nf_pass[tid] = 0u;
        if (tid == 0) {
            st->overflow = 0u;
            st->passes = 0u;
            st->max_nf = (uint32_t)n_roots;
            st->pad = 0u;
        }
    } else {
        s = st->slot[slot];
        if (st->overflow) s.nf = 0u;
        if (s.nf <= limit)
            for (uint32_t k = tid; k < s.nf; k += SQ) fr[0][k] = o.fr[s.buf][k];
    }
    __syncthreads();
    int cur = 0;
    while (s.nf > 0u && s.nf <= limit) {
        // wavefront wv takes entries [e0, e1)
        const uint32_t per = (s.nf + NW * EPW - 1) / (NW * EPW) * EPW;
        const uint32_t e0 = wv * per < s.nf ? wv * per : s.nf, e1 = e0 + per < s.nf ? e0 + per : s.nf;
        U3 c{0u, 0u, 0u};
        for (uint32_t b = e0; b < e1; b += 2 * EPW) {  // two steps' reads in flight
            const uint32_t ea = b + lane / kRun, eb = ea + EPW;
            const int2 pa = fr[cur][ea < e1 ? ea : e0], pb = fr[cur][eb < e1 ? eb : e0];
            const PairRecords ra = load_pair(w, ea < e1, pa, x), rb = load_pair(w, eb < e1, pb, x);
            const int ca = decide(w, ra, x, theta), cb = decide(w, rb, x, theta);
            if (ea < e1) dec[ea * kRun + x] = (int8_t)ca;
            if (eb < e1) dec[eb * kRun + x] = (int8_t)cb;
            U3 unused;
            c = u3add(c, u3add(wave_counts(ca, ra.ta.x & 15, unused), wave_counts(cb, rb.ta.x & 15, unused)));
        }
        if (lane == 0) wtot[wv] = c;
        __syncthreads();
        U3 before{0u, 0u, 0u}, all{0u, 0u, 0u};
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            if (k < wv) before = u3add(before, wtot[k]);
            all = u3add(all, wtot[k]);
        }
        const U3L T{all.a, all.b, all.c};
        if (!pass_fits(o, T, s)) {
            if (tid == 0) st->overflow = 1u;
            s.nf = 0u;
            break;
        }
        int2* nxt = o.fr[s.buf ^ 1u];
        int2* nxt_lds = fr[cur ^ 1];
        auto sink = [&](unsigned long long i, int2 e) {
            nxt[i] = e;
            if (i < kSeqMax) nxt_lds[i] = e;
        };
        unsigned long long on = before.a, of = s.n_far + before.b, onr = s.n_near + before.c;
        for (uint32_t b = e0; b < e1; b += EPW) {
            const uint32_t e = b + lane / kRun;
            const int2 pr = e < e1 ? fr[cur][e] : make_int2(0, 0);
            const int code = e < e1 ? (int)dec[e * kRun + x] : -1;
            const int4 ts = code >= 2 ? w.top[code == 7 ? pr.y : pr.x + x] : make_int4(0, 0, 0, 0);
            U3 lo;
            const U3 k = wave_counts(code, ts.x & 15, lo);
            lane_emit(code, pr.x + x, pr.y, ts, on + lo.a, of + lo.b, onr + lo.c, o.far, o.near, sink);
            on += k.a;
            of += k.b;
            onr += k.c;
        }
        if (tid == 0) pass_done(st, &st->slot[slot ^ 1], s, T);  // the slot is rewritten below
        s = WalkSlot{all.a, s.buf ^ 1u, s.n_far + all.b, s.n_near + all.c};
        cur ^= 1;
        __syncthreads();
    }
    if (tid == 0) st->slot[slot ^ 1] = s;
    if (mb.box) {
        __syncthreads();
        mailbox_write(mb, st, (int)(sizeof(WalkState) / 4));
    }
}

// Larger passes, one launch each.  Workgroup b (by its start ticket) takes a
// contiguous range of entries, each of its wavefronts a contiguous part, so the
// outputs follow the frontier order whatever the grid.  It decides its pairs
// (the decisions and entries kept in LDS, or in memory when the frontier is much
// larger than the grid was sized for), publishes its counts, adds up those of
// the workgroups before it as they appear, and writes its outputs.  It waits only
// for workgroups that have started; a wait past kSpinLimit polls sets the device
// error word.
//
// Bound by latency: the entry, its five records, the counts before it, and then
// the split nodes' records are read one after another.  On 2^20 Plummer particles
// the 18 passes take 308 us; in two launches each, counting and emitting, with
// the decisions through memory, 391 and the gaps between them (steps 3.20 -> 3.08
// ms; 2^20, binary, 1498 -> 1450 us; 100000 particles 756 -> 719).
constexpr int kPassLds = 4;          // entries per thread kept in LDS
constexpr uint32_t kSpinLimit = 1u << 20;
template <int PT>  // threads
__global__ __launch_bounds__(PT) void walk_pass_kernel(WalkNodes w, WalkOut o, WalkState* __restrict__ st, int slot,
                                                       double theta, int8_t* __restrict__ dec,
                                                       PassSync* __restrict__ sync, uint32_t* __restrict__ err) {
    constexpr int NW = PT / kWave, EPW = kWave / kRun, kPassEntries = kPassLds * PT;
    __shared__ int2 ent[kPassEntries];
    __shared__ int8_t code_of[kPassEntries * kRun];
    __shared__ U3 wtot[NW], wbefore[NW];
    __shared__ uint32_t s_b, s_bad;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave, x = lane % kRun;
    if (tid == 0) {
        s_b = atomicAdd(&sync->ticket[slot], 1u);
        s_bad = 0u;
    }
    const WalkSlot s = st->slot[slot];
    const uint32_t nf = st->overflow ? 0u : s.nf;
    __syncthreads();
    const uint32_t b = s_b, G = gridDim.x;
    if (b >= G) return;  // a ticket too many: never, as every pass starts from cleared tickets
    if (tid == 0) {
        for (uint32_t j = b; j < (uint32_t)kPassGrid; j += G) sync->counts[slot ^ 1][j] = 0ull;
        if (b == 0u) sync->ticket[slot ^ 1] = 0u;
    }
    if (nf == 0u) {
        if (b == 0u && tid == 0) st->slot[slot ^ 1] = WalkSlot{0u, s.buf, s.n_far, s.n_near};
        return;
    }
    const int64_t perb = ((int64_t)nf + (int64_t)G * EPW - 1) / ((int64_t)G * EPW) * EPW;
    const int64_t b0 = (int64_t)b * perb < (int64_t)nf ? (int64_t)b * perb : (int64_t)nf;
    const int64_t left = (int64_t)nf - b0;
    const uint32_t n = (uint32_t)(left < perb ? left : perb);
    const bool in_lds = perb <= kPassEntries;
    const int2* fr = o.fr[s.buf] + b0;
    int8_t* decided = dec + b0 * kRun;
    const uint32_t pw = (n + NW * EPW - 1) / (NW * EPW) * EPW;
    const uint32_t e0 = wv * pw < n ? wv * pw : n, e1 = e0 + pw < n ? e0 + pw : n;
    U3 c{0u, 0u, 0u};
    for (uint32_t k = e0; k < e1; k += 2 * EPW) {  // two steps' reads in flight
        const uint32_t ea = k + lane / kRun, eb = ea + EPW;
        const bool va = ea < e1, vb = eb < e1;
        const int2 pa = fr[va ? ea : e0], pb = fr[vb ? eb : e0];
        const PairRecords ra = load_pair(w, va, pa, x), rb = load_pair(w, vb, pb, x);
        const int ca = decide(w, ra, x, theta), cb = decide(w, rb, x, theta);
        if (in_lds) {
            if (va) code_of[ea * kRun + x] = (int8_t)ca;
            if (vb) code_of[eb * kRun + x] = (int8_t)cb;
            if (va && x == 0) ent[ea] = pa;
            if (vb && x == 0) ent[eb] = pb;
        } else {
            if (va) decided[(int64_t)ea * kRun + x] = (int8_t)ca;
            if (vb) decided[(int64_t)eb * kRun + x] = (int8_t)cb;
        }
        U3 unused;
        c = u3add(c, u3add(wave_counts(ca, ra.ta.x & 15, unused), wave_counts(cb, rb.ta.x & 15, unused)));
    }
    if (lane == 0) wtot[wv] = c;
    __syncthreads();
    U3 own{0u, 0u, 0u}, pre{0u, 0u, 0u};  // of the workgroup, of its wavefronts before this one
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        if (k < wv) pre = u3add(pre, wtot[k]);
        own = u3add(own, wtot[k]);
    }
    constexpr unsigned long long kSet = 1ull << 63, kBad = 1ull << 62, kMask = (1ull << kCountBits) - 1ull;
    unsigned long long* counts = sync->counts[slot];
    bool bad = ((own.a | own.b | own.c) >> kCountBits) != 0u;
    if (tid == 0)
        __hip_atomic_store(&counts[b], kSet | (bad ? kBad : (unsigned long long)own.a |
                                                               (unsigned long long)own.b << kCountBits |
                                                               (unsigned long long)own.c << (2 * kCountBits)),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    U3 before{0u, 0u, 0u};
    for (uint32_t j = tid; j < b; j += PT) {
        unsigned long long v;
        uint32_t spins = 0u;
        while (((v = __hip_atomic_load(&counts[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) & kSet) == 0ull) {
            if (++spins > kSpinLimit) {
                atomicOr(err, 1u);
                v = kBad;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        bad |= (v & kBad) != 0ull;
        before = u3add(before, U3{(uint32_t)(v & kMask), (uint32_t)(v >> kCountBits & kMask),
                                  (uint32_t)(v >> (2 * kCountBits) & kMask)});
    }
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1)
        before = u3add(before, U3{(uint32_t)__shfl_xor((int)before.a, d, kWave),
                                  (uint32_t)__shfl_xor((int)before.b, d, kWave),
                                  (uint32_t)__shfl_xor((int)before.c, d, kWave)});
    if (lane == 0) wbefore[wv] = before;
    if (bad) s_bad = 1u;
    __syncthreads();
    before = wbefore[0];
#pragma unroll
    for (int k = 1; k < NW; ++k) before = u3add(before, wbefore[k]);
    // outputs up to this workgroup's: the last one's are the pass's totals
    const U3L T{(unsigned long long)before.a + own.a, (unsigned long long)before.b + own.b,
                (unsigned long long)before.c + own.c};
    const bool fits = s_bad == 0u && pass_fits(o, T, s);
    if (b == G - 1u && tid == 0) {
        if (fits) {
            pass_done(st, &st->slot[slot ^ 1], s, T);
        } else {
            st->overflow = 1u;
            st->slot[slot ^ 1] = WalkSlot{0u, s.buf, s.n_far, s.n_near};
        }
    }
    if (!fits) return;
    int2* nxt = o.fr[s.buf ^ 1u];
    auto sink = [&](unsigned long long i, int2 e) { nxt[i] = e; };
    unsigned long long on = before.a + pre.a, of = s.n_far + before.b + pre.b, onr = s.n_near + before.c + pre.c;
    // a step's split nodes are read while the step before is written
    auto fetch = [&](uint32_t k, int2& pr, int& code) {
        const uint32_t e = k + lane / kRun;
        code = -1;
        pr = make_int2(0, 0);
        if (e < e1) {
            code = in_lds ? code_of[e * kRun + x] : decided[(int64_t)e * kRun + x];
            pr = in_lds ? ent[e] : fr[e];
        }
        return code >= 2 ? w.top[code == 7 ? pr.y : pr.x + x] : make_int4(0, 0, 0, 0);
    };
    int2 pr;
    int code;
    int4 ts = fetch(e0, pr, code);
    for (uint32_t k = e0; k < e1; k += EPW) {
        int2 pr_next;
        int code_next;
        const int4 ts_next = fetch(k + EPW, pr_next, code_next);
        U3 lo;
        const U3 q = wave_counts(code, ts.x & 15, lo);
        lane_emit(code, pr.x + x, pr.y, ts, on + lo.a, of + lo.b, onr + lo.c, o.far, o.near, sink);
        on += q.a;
        of += q.b;
        onr += q.c;
        pr = pr_next;
        code = code_next;
        ts = ts_next;
    }
}

// The same in two launches, for passes of more than kPassMax entries and where the
// host sizes the outputs in between (walk_bfs_sized): the counting kernel decides every pair, stores the decision
// and the block's output counts; the emitting kernel adds the totals of the
// blocks before it and writes the outputs.  Block b of a pass takes a contiguous
// range of tiles of TB / kRun entries.
__device__ __forceinline__ void block_tiles(uint32_t nf, int64_t& t0, int64_t& t1) {
    const int64_t tiles = ((int64_t)nf + TB / kRun - 1) / (TB / kRun);
    const int64_t per = (tiles + gridDim.x - 1) / gridDim.x;
    t0 = (int64_t)blockIdx.x * per;
    t1 = t0 + per < tiles ? t0 + per : tiles;
}

__global__ __launch_bounds__(TB) void walk_count_kernel(WalkNodes w, WalkOut o, const WalkState* __restrict__ st,
                                                        int slot, double theta, int8_t* __restrict__ dec,
                                                        U3L* __restrict__ bsum) {
    __shared__ U3L wsum[TB / kWave];
    const WalkSlot s = st->slot[slot];
    const uint32_t nf = st->overflow ? 0u : s.nf;
    const int2* fr = o.fr[s.buf];
    const int lane = threadIdx.x & (kWave - 1), x = lane % kRun;
    int64_t t0, t1;
    block_tiles(nf, t0, t1);
    U3L c{0ull, 0ull, 0ull};
    for (int64_t t = t0; t < t1; t += 2) {  // two tiles' reads in flight
        const int64_t ia = t * TB + threadIdx.x, ib = ia + TB;
        const int64_t ea = ia / kRun, eb = ib / kRun;
        const bool va = ea < (int64_t)nf, vb = t + 1 < t1 && eb < (int64_t)nf;
        const int2 pa = fr[va ? ea : 0], pb = fr[vb ? eb : 0];
        const PairRecords ra = load_pair(w, va, pa, x), rb = load_pair(w, vb, pb, x);
        const int ca = decide(w, ra, x, theta), cb = decide(w, rb, x, theta);
        if (va) dec[ia] = (int8_t)ca;
        if (vb) dec[ib] = (int8_t)cb;
        U3 unused;
        const U3 k = u3add(wave_counts(ca, ra.ta.x & 15, unused), wave_counts(cb, rb.ta.x & 15, unused));
        if (lane == 0) c = u3ladd(c, k);
    }
    const U3L tot = block_sum(c, wsum);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// Sum of the block totals of a pass (one block), for the host-sized passes.
__global__ __launch_bounds__(TB) void walk_total_kernel(const U3L* __restrict__ bsum, int nb,
                                                        U3L* __restrict__ total) {
    __shared__ U3L wsum[TB / kWave];
    U3L x{0ull, 0ull, 0ull};
    for (int j = threadIdx.x; j < nb; j += TB) x = u3ladd(x, bsum[j]);
    const U3L t = block_sum(x, wsum);
    if (threadIdx.x == 0) *total = t;
}

// Every block sums the block totals itself (the pass total and its own
// offset), so no scan launch sits between counting and emitting.
__global__ __launch_bounds__(TB) void walk_emit_kernel(WalkNodes w, WalkOut o, WalkState* __restrict__ st, int slot,
                                                       const int8_t* __restrict__ dec,
                                                       const U3L* __restrict__ bsum,
                                                       PassSync* __restrict__ sync) {
    constexpr int NW = TB / kWave;
    __shared__ U3L wsum[NW];
    __shared__ U3 wtot[2][NW];
    if (blockIdx.x == 0) {  // for the next pass, as in one launch
        for (int j = threadIdx.x; j < kPassGrid; j += TB) sync->counts[slot ^ 1][j] = 0ull;
        if (threadIdx.x == 0) sync->ticket[slot ^ 1] = 0u;
    }
    const WalkSlot s = st->slot[slot];
    const uint32_t nf = st->overflow ? 0u : s.nf;
    if (nf == 0u) {
        if (blockIdx.x == 0 && threadIdx.x == 0) st->slot[slot ^ 1] = WalkSlot{0u, s.buf, s.n_far, s.n_near};
        return;
    }
    U3L before{0ull, 0ull, 0ull}, all{0ull, 0ull, 0ull};
    for (int j = threadIdx.x; j < (int)gridDim.x; j += TB) {
        const U3L v = bsum[j];
        all = u3ladd(all, v);
        if (j < (int)blockIdx.x) before = u3ladd(before, v);
    }
    const U3L T = block_sum(all, wsum);
    const U3L B = block_sum(before, wsum);
    const bool leader = blockIdx.x == 0 && threadIdx.x == 0;
    if (!pass_fits(o, T, s)) {
        if (leader) {
            st->overflow = 1u;
            st->slot[slot ^ 1] = WalkSlot{0u, s.buf, s.n_far, s.n_near};
        }
        return;
    }
    if (leader) pass_done(st, &st->slot[slot ^ 1], s, T);
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave, x = lane % kRun;
    const int2* fr = o.fr[s.buf];
    int2* nxt = o.fr[s.buf ^ 1u];
    auto sink = [&](unsigned long long i, int2 e) { nxt[i] = e; };
    int64_t t0, t1;
    block_tiles(nf, t0, t1);
    U3L carry{B.a, s.n_far + B.b, s.n_near + B.c};
    // the next tile's entry and decision are read while a tile is written
    auto entry_at = [&](int64_t t, int& code) {
        const int64_t i = t * TB + threadIdx.x, e = i / kRun;
        const bool valid = t < t1 && e < (int64_t)nf;
        code = valid ? (int)dec[i] : -1;
        return fr[valid ? e : 0];
    };
    int code;
    int2 pr = entry_at(t0, code);
    for (int64_t t = t0; t < t1; ++t) {
        int code_next;
        const int2 pr_next = entry_at(t + 1, code_next);
        const int4 ts = code >= 2 ? w.top[code == 7 ? pr.y : pr.x + x] : make_int4(0, 0, 0, 0);
        U3 pre;  // outputs before this lane's, of the tile
        const U3 k = wave_counts(code, ts.x & 15, pre);
        U3* wt = wtot[t & 1];  // the other half is still read by slower wavefronts
        if (lane == 0) wt[wv] = k;
        __syncthreads();
        U3 tot{0u, 0u, 0u};
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            if (q < wv) pre = u3add(pre, wt[q]);
            tot = u3add(tot, wt[q]);
        }
        lane_emit(code, pr.x + x, pr.y, ts, carry.a + pre.a, carry.b + pre.b, carry.c + pre.c, o.far, o.near, sink);
        carry = u3ladd(carry, tot);
        pr = pr_next;
        code = code_next;
    }
}

WalkOut walk_out(Tree& t) {
    const unsigned long long cap = std::min({t.w_fr.cap / 8, t.w_fr2.cap / 8, t.w_dec.cap / kRun, (size_t)UINT32_MAX});
    return WalkOut{{t.w_fr.as<int2>(), t.w_fr2.as<int2>()}, t.m2l_pairs.as<int2>(), t.p2p_pairs.as<int2>(), cap,
                   (unsigned long long)(t.m2l_pairs.cap / 8), (unsigned long long)(t.p2p_pairs.cap / 8)};
}

// mb: the read-back of the state, if this launch is the last before it.
void launch_seq(Tree& t, const WalkNodes& w, int slot, bool init, int limit, double theta, const Mailbox& mb,
                hipStream_t s) {
    hipLaunchKernelGGL(walk_seq_kernel, dim3(1), dim3(SQ), 0, s, w, walk_out(t), t.w_state.as<WalkState>(), slot,
                       init ? 1 : 0, t.n_sets, (uint32_t)limit, theta, t.w_sync.as<PassSync>(), mb);
    TFMM_LAUNCHED();
}

WalkState wait_state(Tree& t, const Mailbox& mb, hipStream_t s) {
    WalkState h;
    // with the device error word: after a wait that ran out the pairs are not
    // all there, and must not be read as lists
    mailbox_wait(t.ctx, mb.seq, sizeof(h), &h, true, s);
    return h;
}

// One pass, for a frontier of about expect entries (any grid covers any
// frontier): smaller workgroups while there are few, so that more compute units
// share the reads, and no more than 256, one per compute unit.  Passes of 500 to
// 2000 entries take 6.4 to 7 us with 256 threads, 7 to 7.5 with 512 and 9 to 10
// with 1024; of 15000 entries 11 to 15, 10 to 11 and 10.5 to 11; of 5e5 43, 37
// and 33 (the workgroups' tickets and counts are in one another's way: 1024
// workgroups take 24 us for any pass).  Past kPassMax entries, whose counts one
// launch could not hand on, two launches.
void launch_pass(Tree& t, const WalkNodes& w, int slot, int64_t expect, double theta, hipStream_t s) {
    if (expect > kPassMax) {
        t.w_off.ensure(t.ctx, (size_t)kWalkGrid * sizeof(U3L));
        hipLaunchKernelGGL(walk_count_kernel, dim3(kWalkGrid), dim3(TB), 0, s, w, walk_out(t),
                           (const WalkState*)t.w_state.as<WalkState>(), slot, theta, t.w_dec.as<int8_t>(),
                           t.w_off.as<U3L>());
        TFMM_LAUNCHED();
        hipLaunchKernelGGL(walk_emit_kernel, dim3(kWalkGrid), dim3(TB), 0, s, w, walk_out(t),
                           t.w_state.as<WalkState>(), slot, (const int8_t*)t.w_dec.as<int8_t>(),
                           (const U3L*)t.w_off.as<U3L>(), t.w_sync.as<PassSync>());
        TFMM_LAUNCHED();
        return;
    }
    auto run = [&](auto kern, int threads) {
        const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>(kPassGrid, cdiv(expect, threads / kRun)));
        hipLaunchKernelGGL(kern, dim3(g), dim3(threads), 0, s, w, walk_out(t), t.w_state.as<WalkState>(), slot, theta,
                           t.w_dec.as<int8_t>(), t.w_sync.as<PassSync>(), t.ctx->dev_err);
        TFMM_LAUNCHED();
    };
    if (expect <= 2048) run(walk_pass_kernel<256>, 256);
    else if (expect <= 16384) run(walk_pass_kernel<512>, 512);
    else run(walk_pass_kernel<1024>, 1024);
}

// Frontier passes sized on the host: the totals of every pass are read back
// and the buffers grown before its outputs are written.  Used whenever the
// unsynchronised passes run out of room.
void walk_bfs_sized(Tree& t, const WalkNodes& w, double theta, hipStream_t s) {
    Ctx* ctx = t.ctx;
    const int64_t nn = t.n_nodes;
    int64_t cap_far = (int64_t)(t.m2l_pairs.cap / 8), cap_near = (int64_t)(t.p2p_pairs.cap / 8);
    if (cap_far < 4096) {
        cap_far = std::max<int64_t>(4096, 64 * nn);
        t.m2l_pairs.ensure(ctx, (size_t)cap_far * 8);
    }
    if (cap_near < 4096) {
        cap_near = std::max<int64_t>(4096, 16 * nn);
        t.p2p_pairs.ensure(ctx, (size_t)cap_near * 8);
    }
    t.w_fr.ensure(ctx, (size_t)std::max(4096, t.n_sets) * 8);
    t.w_fr2.ensure(ctx, (size_t)std::max(4096, t.n_sets) * 8);
    t.w_off.ensure(ctx, (size_t)kWalkGrid * sizeof(U3L));
    t.w_dec.ensure(ctx, (size_t)std::max(4096, t.n_sets) * kRun);
    t.w_state.ensure(ctx, sizeof(WalkState));
    t.w_sync.ensure(ctx, sizeof(PassSync));
    t.scratch2.ensure(ctx, 256);
    WalkState* st = t.w_state.as<WalkState>();
    U3L* tot = t.scratch2.as<U3L>();
    launch_seq(t, w, 1, true, 0, theta, Mailbox{}, s);  // the roots, into slot 0 and buffer 0
    int64_t nf = t.n_sets, max_nf = t.n_sets, n_far = 0, n_near = 0;
    int slot = 0;
    t.walk_hint_nf.clear();
    for (int k = 0; nf > 0; ++k) {
        t.walk_hint_nf.push_back(nf);
        const unsigned g = (unsigned)std::min<int64_t>(kWalkGrid, cdiv(nf, TB / kRun));
        DevBuf& nxt = (k & 1) ? t.w_fr : t.w_fr2;
        // buffers resized here are idle: a resize waits for the device
        t.w_dec.ensure(ctx, (size_t)nf * kRun);
        hipLaunchKernelGGL(walk_count_kernel, dim3(g), dim3(TB), 0, s, w, walk_out(t), (const WalkState*)st, slot,
                           theta, t.w_dec.as<int8_t>(), t.w_off.as<U3L>());
        TFMM_LAUNCHED();
        hipLaunchKernelGGL(walk_total_kernel, dim3(1), dim3(TB), 0, s, (const U3L*)t.w_off.as<U3L>(), (int)g, tot);
        TFMM_LAUNCHED();
        const U3L T = read_back(ctx, (const U3L*)tot, s);
        if (T.a > UINT32_MAX || T.b > UINT32_MAX || T.c > UINT32_MAX)
            fail(TFMM_ENOMEM, "walk: one frontier pass would emit more than 2^32 pairs");
        if (n_far + (int64_t)T.b > cap_far) {
            cap_far = std::max<int64_t>(2 * cap_far, n_far + (int64_t)T.b);
            t.m2l_pairs.ensure_keep(ctx, (size_t)cap_far * 8, s);
        }
        if (n_near + (int64_t)T.c > cap_near) {
            cap_near = std::max<int64_t>(2 * cap_near, n_near + (int64_t)T.c);
            t.p2p_pairs.ensure_keep(ctx, (size_t)cap_near * 8, s);
        }
        nxt.ensure(ctx, (size_t)std::max<unsigned long long>(T.a, 1) * 8);
        WalkOut o = walk_out(t);
        o.cap_next = std::min<size_t>(nxt.cap / 8, UINT32_MAX);  // the decisions grow before the next count
        hipLaunchKernelGGL(walk_emit_kernel, dim3(g), dim3(TB), 0, s, w, o, st, slot,
                           (const int8_t*)t.w_dec.as<int8_t>(), (const U3L*)t.w_off.as<U3L>(),
                           t.w_sync.as<PassSync>());
        TFMM_LAUNCHED();
        n_far += (int64_t)T.b;
        n_near += (int64_t)T.c;
        nf = (int64_t)T.a;
        max_nf = std::max(max_nf, nf);
        slot ^= 1;
    }
    const WalkState h = read_back(ctx, (const WalkState*)st, s);
    if (h.overflow)
        fail(TFMM_EDEVICE, "walk: a host-sized frontier pass reported an overflow");
    t.n_m2l = n_far;
    t.n_p2p = n_near;
    t.walk_hint_fr = max_nf;
}

// Room for the lists of a tree's first walk: far and near pairs and frontier
// entries per node grow like (1 + 2 / theta)^3, the volume within 1 / theta
// cell sizes (ball, Plummer and disk sets of 10^3 to 10^6 particles, theta 0.2 to
// 0.95: far up to 1.6, near up to 0.75, frontier up to about 0.05 of it per
// node).  A walk that needs more runs the host-sized passes, and so does one for
// which the estimate does not fit the memory there is.
void first_room(const Tree& t, const std::vector<double>& theta, int64_t& fr, int64_t& far, int64_t& near) {
    const double th = std::max(*std::min_element(theta.begin(), theta.end()), 0.05);
    const double around = (1.0 + 2.0 / th) * (1.0 + 2.0 / th) * (1.0 + 2.0 / th);
    const double nn = (double)t.n_nodes, all = 0.5 * nn * (nn + 1.0);
    far = (int64_t)std::min(all, nn * std::min(1.65 * around, 400.0)) + 4096;
    near = (int64_t)std::min(all, nn * std::min(0.75 * around + 8.0, 160.0)) + 4096;
    fr = (int64_t)std::min(all, nn * std::min(0.06 * around + 2.0, 32.0)) + 4096 + t.n_sets;
}

// Under a budget the surplus of a first walk's estimate goes back to the context,
// where other trees may need it.  If there is no memory for that, it stays.
void fit_room(Tree& t, hipStream_t s) {
    try {
        const size_t fr = (size_t)(t.walk_hint_fr + t.walk_hint_fr / 4 + 4096);
        for (DevBuf* b : {&t.w_fr, &t.w_fr2, &t.w_dec}) b->fit(fr * 8, s);
        t.m2l_pairs.fit((size_t)t.n_m2l * 8, s);
        t.p2p_pairs.fit((size_t)t.n_p2p * 8, s);
        t.walk_estimated = false;
    } catch (const Error& e) {
        if (e.code != TFMM_ENOMEM) throw;
    }
}

// Frontier passes with no host synchronisation, sized from the previous walk
// of this tree plus a quarter: the first passes, while they are small, in one
// launch, then a launch per pass as many as that walk had larger ones, then
// the last small passes in one launch.  The host reads the state back once; a
// frontier that is left (the passes came out differently) gets more launches.
// A tree's first walk reads the state back after the first launch too, and its
// room is estimated.  Returns false (lists invalid) when the host-sized passes
// must be used instead.
bool walk_bfs_async(Tree& t, const WalkNodes& w, const std::vector<double>& thetas, hipStream_t s,
                    const std::function<void()>& queued) {
    Ctx* ctx = t.ctx;
    const double theta = thetas[0];
    const bool known = t.walk_hint_fr > 0;
    int64_t want_fr, want_far, want_near;
    if (known) {
        want_fr = t.walk_hint_fr + t.walk_hint_fr / 4 + 4096;
        want_far = t.walk_hint_far + t.walk_hint_far / 4 + 4096;
        want_near = t.walk_hint_near + t.walk_hint_near / 4 + 4096;
    } else {
        if (t.walk_sized) return false;
        first_room(t, thetas, want_fr, want_far, want_near);
        const int64_t bytes = 8 * (4 * want_fr + want_far + want_near);
        if (ctx->budget && ctx->used - ctx->cached + (size_t)bytes > ctx->budget / 2) return false;
    }
    if (want_fr > (int64_t)UINT32_MAX) return false;
    t.w_state.ensure(ctx, sizeof(WalkState));
    t.w_sync.ensure(ctx, sizeof(PassSync));
    try {
        t.w_fr.ensure(ctx, (size_t)want_fr * 8);
        t.w_fr2.ensure(ctx, (size_t)want_fr * 8);
        t.w_dec.ensure(ctx, (size_t)want_fr * kRun);
        t.m2l_pairs.ensure(ctx, (size_t)want_far * 8);
        t.p2p_pairs.ensure(ctx, (size_t)want_near * 8);
    } catch (const Error& e) {
        if (known || e.code != TFMM_ENOMEM) throw;
        drop_walk_room(t);
        return false;
    }
    if (!known) t.walk_estimated = true;
    int slot = 0;
    // larger passes of the previous walk: from the first above the limit to the last
    int a = 0, b = (int)t.walk_hint_nf.size();
    if (!known || t.walk_hint_fr <= kSeqHead) b = 0;
    const int limit = b > 0 ? kSeqEnds : kSeqHead;
    while (a < b && t.walk_hint_nf[a] <= limit) ++a;
    while (b > a && t.walk_hint_nf[b - 1] <= limit) --b;
    const Mailbox mb = mailbox_next(ctx);
    launch_seq(t, w, slot ^ 1, true, limit, theta, b > a ? Mailbox{} : mb, s);
    if (b > a) {
        for (int k = a; k < b; ++k, slot ^= 1)
            launch_pass(t, w, slot, t.walk_hint_nf[k] + t.walk_hint_nf[k] / 4 + 64, theta, s);
        launch_seq(t, w, slot, false, kSeqMax, theta, mb, s);
        slot ^= 1;
    }
    queued();
    WalkState h = wait_state(t, mb, s);
    while (!h.overflow && h.slot[slot].nf != 0u) {
        if (h.passes > (uint32_t)kMaxPasses) return false;
        const int64_t nf = h.slot[slot].nf;
        for (int k = 0; k < 4; ++k, slot ^= 1) launch_pass(t, w, slot, nf << k, theta, s);
        const Mailbox more = mailbox_next(ctx);
        launch_seq(t, w, slot, false, kSeqMax, theta, more, s);
        slot ^= 1;
        h = wait_state(t, more, s);
    }
    if (h.overflow) return false;
    t.n_m2l = (int64_t)h.slot[slot].n_far;
    t.n_p2p = (int64_t)h.slot[slot].n_near;
    t.walk_hint_fr = h.max_nf;
    t.walk_hint_nf.assign(h.nf_pass, h.nf_pass + std::min<uint32_t>(h.passes, (uint32_t)kMaxPasses));
    if (t.walk_estimated && ctx->budget) fit_room(t, s);
    return true;
}

}  // namespace

void drop_walk_room(Tree& t) {
    for (DevBuf* b : {&t.w_fr, &t.w_fr2, &t.w_dec, &t.m2l_pairs, &t.p2p_pairs}) b->release();
    t.walk_valid = false;
    t.walk_estimated = false;
    t.walk_sized = true;
}

// Fork the tree's second stream from s / join it back into s.
void aux_fork(Tree& t, hipStream_t s) {
    if (!t.aux) {
        TFMM_HIP(hipStreamCreateWithFlags(&t.aux, hipStreamNonBlocking));
        TFMM_HIP(hipEventCreateWithFlags(&t.fork_ev, hipEventDisableTiming));
        TFMM_HIP(hipEventCreateWithFlags(&t.join_ev, hipEventDisableTiming));
    }
    TFMM_HIP(hipEventRecord(t.fork_ev, s));
    TFMM_HIP(hipStreamWaitEvent(t.aux, t.fork_ev, 0));
}

void aux_join(Tree& t, hipStream_t s) {
    TFMM_HIP(hipEventRecord(t.join_ev, t.aux));
    TFMM_HIP(hipStreamWaitEvent(s, t.join_ev, 0));
}

// The frontier passes on s, then the far-list chain on the tree's second
// stream (after the passes) and the near-list chain on s.  walk_lists_end
// reads the totals back once the near chain is done.
void walk_lists_begin(Tree& t, const std::vector<double>& theta_in, hipStream_t s, hipEvent_t passes_done,
                      const std::function<void()>& meanwhile, bool near_first) {
    const int64_t nn = t.n_nodes;
    if (theta_in.size() != 1 && theta_in.size() != (size_t)t.n_sets) fail(TFMM_EINVAL, "theta: one value or one per set");
    const std::vector<double> theta_keep = theta_in;  // the caller's vector may be the tree's own
    const double theta = theta_keep[0];
    const double* theta_dev = nullptr;
    if (theta_keep.size() > 1) {
        upload(t, t.set_theta, theta_keep.data(), theta_keep.size() * sizeof(double), 1, s);
        theta_dev = t.set_theta.as<double>();
    }
    WalkNodes w{t.w_geo.as<double4>(), t.w_top.as<int4>(), theta_dev, (int32_t)nn};
    t.walk_valid = false;
    bool called = false;
    const std::function<void()> once = [&] {
        if (!called) meanwhile();
        called = true;
    };
    if (!walk_bfs_async(t, w, theta_keep, s, once)) {
        once();
        walk_bfs_sized(t, w, theta, s);
    }
    t.walk_hint_far = t.n_m2l;
    t.walk_hint_near = t.n_p2p;
    if (passes_done) TFMM_HIP(hipEventRecord(passes_done, s));
    if (!lists_fit(t.n_m2l, t.n_p2p))
        fail(TFMM_ENOMEM, "walk: " + std::to_string(t.n_m2l) + " far and " + std::to_string(t.n_p2p) +
                              " near pairs exceed the lists' 32-bit offsets");

    // The far-list chain runs on the tree's second stream, the near-list chain
    // on s; they share no buffer.
    aux_fork(t, s);
    if (near_first) build_near_lists(t, s);
    build_far_lists(t, t.aux);
    if (!near_first) build_near_lists(t, s);
    t.walk_theta = theta_keep;
}

void walk_lists_end(Tree& t, hipStream_t s) {
    near_lists_end(t, s);
    t.walk_valid = true;
}

void walk_tree(Tree& t, const std::vector<double>& theta, hipStream_t s) {
    Unfinished work(t, s);
    walk_lists_begin(t, theta, s, nullptr, [] {}, false);
    aux_join(t, s);
    walk_lists_end(t, s);
    work.done = true;
}

}  // namespace tfmm
