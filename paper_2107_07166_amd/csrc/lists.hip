// Per-target interaction lists from the walk's pairs.
//
// A list holds the sources of one target node in the walk's emission order
// (the interaction kernels sum in list order, so the order is part of the
// result).  The directed entries of the pairs (both ways; a near self pair
// once) are grouped by target in two steps:
//   1. one stable partition into at most 1024 buckets of targets (counts per
//      tile and bucket, a scan over them, a ranked scatter through LDS);
//   2. one workgroup per bucket counts its targets, places its entries, and
//      writes the list bounds; for the near lists also the running source count
//      along the lists and each target's number of work items.
// Bucket of a target: its high bits for the far lists, which M2L reads as one
// array of consecutive lists; its low bits for the near lists, so that the
// long lists of the shallow leaves of a sparse halo (neighbours in node order,
// up to 30 % of all near entries on 2^18 Plummer particles) land in different
// buckets.  An entry is one word, (target << 16) | source, when node ids fit 16
// bits, else two.  Against sorting the entries by all target bits, in two or
// three passes, and deriving the bounds and prefixes in launches of their own,
// this reads and writes them half as often and takes a third of the launches:
// a solve of 2^11 particles 253 -> 223 us, of 2^18 1665 -> 1625 us, of 2^22
// 6.83 -> 6.61 ms (disk, order 6; 2^20 Plummer particles, where the near lists of
// the halo hold one workgroup up, 3.19 ms both).
#include <algorithm>
#include <cstddef>

#include "common.h"
#include "list_math.h"

namespace tfmm {
namespace {

constexpr int TB = 256;

__global__ __launch_bounds__(TB) void fill_i32_kernel(int32_t* __restrict__ p, int64_t n, int32_t v) {
    const int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x;
    if (i < n) p[i] = v;
}

unsigned grid(int64_t n) { return (unsigned)cdiv(n > 0 ? n : 1, TB); }

int bits_for(int64_t n) {
    int b = 1;
    while (((int64_t)1 << b) < n) ++b;
    return b;
}

// Device slots of the list-building totals, read back together at the end.
struct WalkTotals {
    uint32_t multi;        // leaves split into several near-field items
    uint32_t near_entries; // directed near entries (check of 2 n_near - n_leaves)
    uint32_t items;        // near-field work items
    uint32_t partial;      // partial-sum rows of multi-item leaves, mod 2^32
    unsigned long long rows;  // all of them
    uint32_t scratch[12];  // totals nobody reads
    unsigned long long near_int;
};

// ---- partition into buckets ------------------------------------------------------
constexpr int PB = 512;                  // threads of a partition tile
constexpr int PW = PB / kWave;
constexpr int PI = 16;                   // entries per thread
constexpr int PT = PB * PI;              // entries per tile
constexpr int kBucketBits = 10;
constexpr int NBK = 1 << kBucketBits;    // most buckets
constexpr int kRows = 64;                // tiles whose counts are scanned together
constexpr int64_t kDirectRows = 64;      // up to this many tiles: one scan over all

template <typename Word> struct WordBits;
template <> struct WordBits<uint32_t> { static constexpr int src = 16; };
template <> struct WordBits<uint64_t> { static constexpr int src = 32; };

// near: a target's low `bits` bits pick its bucket, else the bits above `shift`.
struct Split {
    int near, bits, shift;
    __device__ __forceinline__ uint32_t bucket(uint32_t t) const {
        return near ? (t & ((1u << bits) - 1u)) : (t >> shift);
    }
    __device__ __forceinline__ uint32_t local(uint32_t t) const {
        return near ? (t >> bits) : (t & ((1u << shift) - 1u));
    }
    __device__ __forceinline__ uint32_t target(uint32_t b, uint32_t l) const {
        return near ? ((l << bits) | b) : ((b << shift) | l);
    }
};

// Entry i of the pairs, target and source; false past the end and for the
// second half of a self pair.
__device__ __forceinline__ bool entry(const int2* __restrict__ pairs, int64_t ne, int64_t i, uint32_t& t,
                                      uint32_t& s) {
    t = s = 0u;
    if (i >= ne) return false;
    const int2 q = pairs[i >> 1];
    t = (uint32_t)((i & 1) ? q.y : q.x);
    s = (uint32_t)((i & 1) ? q.x : q.y);
    return !((i & 1) && q.x == q.y);
}

// Counts of a tile's buckets, cnt[tile][bucket].
__global__ __launch_bounds__(PB) void bucket_count_kernel(const int2* __restrict__ pairs, int64_t ne, Split sp, int nb,
                                                          uint32_t* __restrict__ cnt) {
    __shared__ uint32_t h[NBK];
    for (int d = threadIdx.x; d < NBK; d += PB) h[d] = 0u;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * PT + threadIdx.x;
#pragma unroll 4
    for (int r = 0; r < PI; ++r) {
        uint32_t t, unused;
        if (entry(pairs, ne, i0 + r * PB, t, unused)) atomicAdd(&h[sp.bucket(t)], 1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < nb; d += PB) cnt[(int64_t)blockIdx.x * nb + d] = h[d];
}

// Prefixes over kRows tiles of every bucket's counts, in place, and their totals.
__global__ __launch_bounds__(TB) void bucket_rows_kernel(uint32_t* __restrict__ cnt, int64_t rows, int nb,
                                                         uint32_t* __restrict__ tot) {
    const int d = blockIdx.y * TB + threadIdx.x;
    if (d >= nb) return;
    const int64_t r0 = (int64_t)blockIdx.x * kRows, r1 = r0 + kRows < rows ? r0 + kRows : rows;
    uint32_t run = 0u;
    for (int64_t r = r0; r < r1; r += 8) {
        uint32_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = r + u < r1 ? cnt[(r + u) * nb + d] : 0u;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (r + u < r1) cnt[(r + u) * nb + d] = run;
            run += x[u];
        }
    }
    tot[(int64_t)blockIdx.x * nb + d] = run;
}

// Exclusive scan over PB threads' values (two per thread in order a, b); every
// thread calls it.
__device__ __forceinline__ uint32_t block_excl(uint32_t v, uint32_t* wsum, uint32_t& total) {
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave, nw = blockDim.x / kWave;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t u = (uint32_t)__shfl_up((int)incl, o, kWave);
        if (lane >= o) incl += u;
    }
    if (lane == kWave - 1) wsum[wv] = incl;
    __syncthreads();
    uint32_t off = 0u, all = 0u;
    for (int k = 0; k < nw; ++k) {
        if (k < wv) off += wsum[k];
        all += wsum[k];
    }
    __syncthreads();
    total = all;
    return off + incl - v;
}

// Bucket starts: M[row][bucket] (counts, or totals of kRows tiles) becomes the
// place of the row's first entry of the bucket; start[nb] is the entry count
// (for the near lists also in their totals res).  One block, a thread per bucket.
__global__ __launch_bounds__(NBK) void bucket_starts_kernel(uint32_t* __restrict__ M, int64_t rows, int nb,
                                                            uint32_t* __restrict__ start,
                                                            WalkTotals* __restrict__ res) {
    __shared__ uint32_t wsum[NBK / kWave];
    const int d = threadIdx.x;
    uint32_t sum = 0u;
    if (d < nb)
        for (int64_t r = 0; r < rows; r += 8) {
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (r + u < rows) sum += M[(r + u) * nb + d];
        }
    uint32_t all;
    uint32_t run = block_excl(sum, wsum, all);
    if (d < nb) {
        start[d] = run;
        for (int64_t r = 0; r < rows; r += 8) {
            uint32_t x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = r + u < rows ? M[(r + u) * nb + d] : 0u;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (r + u < rows) M[(r + u) * nb + d] = run;
                run += x[u];
            }
        }
    }
    if (d == 0) {
        start[nb] = all;
        if (res) {
            res->near_entries = all;
            res->multi = 0u;
            res->rows = 0ull;
        }
    }
}

__device__ __forceinline__ uint64_t lanes_below() {
    const int lane = threadIdx.x & (kWave - 1);
    return lane == 0 ? 0ull : (~0ull >> (kWave - lane));
}

// Scatters a tile's entries into the buckets, in order.  A single tile (cnt ==
// nullptr && M == nullptr) finds the starts itself.
template <typename Word>
__global__ __launch_bounds__(PB) void bucket_scatter_kernel(const int2* __restrict__ pairs, int64_t ne, Split sp,
                                                            int nb, const uint32_t* __restrict__ cnt,
                                                            const uint32_t* __restrict__ M, int rows_per,
                                                            Word* __restrict__ out, uint32_t* __restrict__ start,
                                                            WalkTotals* __restrict__ res) {
    __shared__ uint16_t wc[PW][NBK];
    __shared__ uint32_t gbase[NBK];
    __shared__ uint16_t dstart[NBK];
    __shared__ uint32_t wsum[PW];
    __shared__ Word st[PT];
    constexpr int SB = WordBits<Word>::src;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int64_t tile = blockIdx.x;
    for (int d = lane; d < NBK; d += kWave) wc[wv][d] = 0;
    if (M)
        for (int d = tid; d < nb; d += PB)
            gbase[d] = M[(tile / rows_per) * nb + d] + (cnt ? cnt[tile * nb + d] : 0u);
    const int64_t i0 = tile * PT + (int64_t)wv * (kWave * PI) + lane;
    uint32_t tg[PI], sr[PI];
    uint16_t rank[PI];
    uint32_t ok = 0u;
#pragma unroll
    for (int r = 0; r < PI; ++r)
        if (entry(pairs, ne, i0 + r * kWave, tg[r], sr[r])) ok |= 1u << r;
    const uint64_t lt = lanes_below();
#pragma unroll
    for (int r = 0; r < PI; ++r) {
        const bool valid = (ok >> r) & 1u;
        const uint32_t d = sp.bucket(tg[r]);
        const uint64_t peers = same_lanes(valid, d, sp.bits);
        const int below = __popcll(peers & lt);
        rank[r] = 0;
        if (valid) {
            const uint16_t first = wc[wv][d];
            rank[r] = (uint16_t)(first + below);
            if (below == 0) wc[wv][d] = (uint16_t)(first + __popcll(peers));
        }
    }
    __syncthreads();
    // per bucket: offsets of the wavefronts; then of the buckets in the tile
    constexpr int DPT = NBK / PB;
    uint32_t tot[DPT], sum = 0u;
#pragma unroll
    for (int k = 0; k < DPT; ++k) {
        const int d = tid * DPT + k;
        uint32_t t = 0u;
#pragma unroll
        for (int q = 0; q < PW; ++q) {
            const uint32_t c = wc[q][d];
            wc[q][d] = (uint16_t)t;
            t += c;
        }
        tot[k] = t;
        sum += t;
    }
    uint32_t nvalid;
    uint32_t run = block_excl(sum, wsum, nvalid);
#pragma unroll
    for (int k = 0; k < DPT; ++k) {
        const int d = tid * DPT + k;
        dstart[d] = (uint16_t)run;
        if (!M) {
            gbase[d] = run;
            if (d <= nb) start[d] = run;
        }
        run += tot[k];
    }
    if (!M && tid == 0) {
        start[nb] = nvalid;
        if (res) {
            res->near_entries = nvalid;
            res->multi = 0u;
            res->rows = 0ull;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PI; ++r) {
        if (!((ok >> r) & 1u)) continue;
        const uint32_t d = sp.bucket(tg[r]);
        st[dstart[d] + wc[wv][d] + rank[r]] = ((Word)tg[r] << SB) | (Word)sr[r];
    }
    __syncthreads();
    for (uint32_t i = tid; i < nvalid; i += PB) {
        const Word x = st[i];
        const uint32_t d = sp.bucket((uint32_t)(x >> SB));
        out[gbase[d] + (i - dstart[d])] = x;
    }
}

// What the near lists need besides their bounds: the sources before every
// entry along its bucket (as source_step counts them, mod 2^32), and per target
// its items and partial rows.
struct NearOut {
    const int32_t* count;
    uint32_t *P, *nitems, *prows;
};

// Items and partial-sum rows (mod 2^32) of a target leaf's list.
__device__ __forceinline__ void leaf_items(const uint32_t* P, uint32_t q0, uint32_t q1, int32_t count, uint32_t* nit,
                                           uint32_t* prw) {
    const uint32_t n = list_items(P, q0, q1);
    *nit = n;
    *prw = (uint32_t)item_rows(n, count);
}

// One bucket: its targets' lists.  l0[t], l1[t]: the list of target t is src
// entries [l0, l1).  FAR: l0 is the offset array (l1 = l0 + 1; its last element
// is written by the last bucket).  lbits: bits of a target's place in the bucket.
// Bound by the serial passes of the workgroup whose bucket holds the longest
// lists.  512 threads: with 1024 that bucket ends sooner (the near lists of 2^20
// Plummer particles 105 us alone instead of 118), but a solve, where it runs
// beside the other chain, gained nothing there (3.19 ms both) and lost 3 % on a
// binary of 2^20 (1579 us, 1516 with 512).
constexpr int LT = 512;                  // threads of the workgroup
constexpr int LW = LT / kWave;
constexpr int LTILE = LT * PI;           // entries placed together
constexpr int kLocalBits = 9;
constexpr int NLB = 1 << kLocalBits;     // most targets of a bucket
constexpr int LP = 8;                    // entries per thread of the prefix
static_assert(LTILE <= (int)kListStep && 8 * LT <= (int)kListStep, "loops over the entries end");
template <typename Word, bool NEAR>
__global__ __launch_bounds__(LT) void bucket_lists_kernel(const Word* __restrict__ in,
                                                          const uint32_t* __restrict__ start, Split sp, int nb,
                                                          int lbits, int64_t nn, uint32_t* __restrict__ src,
                                                          uint32_t* __restrict__ l0, uint32_t* __restrict__ l1,
                                                          NearOut no) {
    __shared__ uint16_t wc[LW][NLB];
    __shared__ uint32_t pos[NLB];                        // next place of every target's list
    __shared__ uint32_t wsum[LW];
    __shared__ uint32_t st[NEAR ? LT * (LP + 1) : 1];    // values of the prefix
    constexpr int SB = WordBits<Word>::src;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const uint32_t b = blockIdx.x;
    const uint32_t E0 = start[b], E1 = start[b + 1];
    const int nl = 1 << lbits;  // places of the bucket (some past the last node)
    for (int d = tid; d < nl; d += LT) pos[d] = 0u;
    __syncthreads();
    for (uint32_t q0 = E0; q0 < E1; q0 += 8 * LT) {
        Word x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t q = q0 + u * LT + tid;
            x[u] = in[q < E1 ? q : E0];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool valid = q0 + u * LT + tid < E1;
            const uint32_t d = sp.local((uint32_t)(x[u] >> SB));
            const uint64_t vm = __ballot(valid);
            if (vm == 0ull) break;
            // a long list fills whole wavefronts with one target: one addition
            const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
            if (__ballot(valid && d != d0) == 0ull) {
                if (lane == 0) atomicAdd(&pos[d0], (uint32_t)__popcll(vm));
            } else if (valid) {
                atomicAdd(&pos[d], 1u);
            }
        }
    }
    __syncthreads();
    static_assert(NLB <= LT, "a thread per place");
    {
        const uint32_t tot = tid < nl ? pos[tid] : 0u;
        uint32_t unused;
        const uint32_t run = E0 + block_excl(tot, wsum, unused);
        if (tid < nl) {
            const int64_t t = sp.target(b, (uint32_t)tid);
            pos[tid] = run;
            if (t < nn) {
                l0[t] = run;
                if (NEAR) l1[t] = run + tot;
            }
        }
    }
    if (!NEAR && b == (uint32_t)nb - 1u && tid == 0) l0[nn] = E1;
    const uint64_t lt = lanes_below();
    for (uint32_t q0 = E0; q0 < E1; q0 += LTILE) {
        for (int d = lane; d < nl; d += kWave) wc[wv][d] = 0;
        __syncthreads();
        const uint32_t i0 = q0 + wv * (kWave * PI) + lane;
        Word w[PI];
        uint16_t rank[PI];
#pragma unroll
        for (int r = 0; r < PI; ++r) w[r] = i0 + r * kWave < E1 ? in[i0 + r * kWave] : (Word)0;
#pragma unroll
        for (int r = 0; r < PI; ++r) {
            const bool valid = i0 + r * kWave < E1;
            rank[r] = 0;
            if (__ballot(valid) == 0ull) break;
            const uint32_t d = sp.local((uint32_t)(w[r] >> SB));
            const uint64_t peers = same_lanes(valid, d, lbits);
            const int below = __popcll(peers & lt);
            if (valid) {
                const uint16_t first = wc[wv][d];
                rank[r] = (uint16_t)(first + below);
                if (below == 0) wc[wv][d] = (uint16_t)(first + __popcll(peers));
            }
        }
        __syncthreads();
        uint32_t add = 0u;
        if (tid < nl) {
#pragma unroll
            for (int x = 0; x < LW; ++x) {
                const uint32_t c = wc[x][tid];
                wc[x][tid] = (uint16_t)add;
                add += c;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < PI; ++r) {
            if (i0 + r * kWave >= E1) continue;
            const uint32_t d = sp.local((uint32_t)(w[r] >> SB));
            src[pos[d] + wc[wv][d] + rank[r]] = (uint32_t)(w[r] & (((Word)1 << SB) - 1));
        }
        __syncthreads();
        if (tid < nl) pos[tid] += add;
        __syncthreads();
    }
    if constexpr (NEAR) {
        uint32_t carry = 0u;
        for (uint32_t q0 = E0; q0 < E1; q0 += LT * LP) {
            // read and written striped, scanned by consecutive runs, through LDS
#pragma unroll
            for (int r = 0; r < LP; ++r) {
                const uint32_t i = r * LT + tid;
                st[i + i / LP] = q0 + i < E1 ? source_step(no.count[src[q0 + i]]) : 0u;
            }
            __syncthreads();
            uint32_t c[LP], sumc = 0u;
#pragma unroll
            for (int r = 0; r < LP; ++r) {
                c[r] = st[tid * (LP + 1) + r];
                sumc += c[r];
            }
            uint32_t all;
            uint32_t p = carry + block_excl(sumc, wsum, all);
#pragma unroll
            for (int r = 0; r < LP; ++r) {
                st[tid * (LP + 1) + r] = p;
                p += c[r];
            }
            carry += all;
            __syncthreads();
#pragma unroll
            for (int r = 0; r < LP; ++r) {
                const uint32_t i = r * LT + tid;
                if (q0 + i < E1) no.P[q0 + i] = st[i + i / LP];
            }
            __syncthreads();
        }
        __syncthreads();
        if (tid < nl) {
            const int64_t t = sp.target(b, (uint32_t)tid);
            if (t < nn) leaf_items(no.P, l0[t], l1[t], no.count[t], &no.nitems[t], &no.prows[t]);
        }
    }
}

// ---- large trees: sorts by all target bits -----------------------------------------
// CSR offsets from targets sorted ascending:
// off[t] = first entry with target >= t, for t = 0..nn.  Entry boundary i
// (0..ne) writes off[t] for targets t in (target[i-1], target[i]], so each t
// is written by exactly one boundary, which also copies off[nn] (the number
// of entries below nn) to *below_nn if given.  Targets may equal nn (entries
// sorted after every real one).  A thread takes four boundaries and reads
// their keys with one 16-byte load.
__global__ __launch_bounds__(TB) void csr_offsets_kernel(const uint32_t* __restrict__ keys, int64_t ne,
                                                         int64_t nn, uint32_t* __restrict__ off,
                                                         uint32_t* __restrict__ below_nn) {
    const int64_t i0 = ((int64_t)blockIdx.x * TB + threadIdx.x) * 4;
    if (i0 > ne) return;
    int64_t kv[5];  // targets of entries i0 - 1 .. i0 + 3 (-1 before the first, nn after the last)
    kv[0] = i0 == 0 ? -1 : (int64_t)keys[i0 - 1];
    if (i0 + 4 <= ne) {
        const uint4 q = *reinterpret_cast<const uint4*>(keys + i0);
        kv[1] = q.x;
        kv[2] = q.y;
        kv[3] = q.z;
        kv[4] = q.w;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) kv[j + 1] = i0 + j < ne ? (int64_t)keys[i0 + j] : nn;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int64_t i = i0 + j;
        if (i > ne) break;
        const int64_t lo = kv[j] + 1;
        const int64_t hi = kv[j + 1] < nn ? kv[j + 1] : nn;
        for (int64_t t = lo; t <= hi; ++t) off[t] = (uint32_t)i;
        if (below_nn && lo <= nn && nn <= hi) *below_nn = (uint32_t)i;
    }
}

// Items of every node's near list from offsets.
__global__ __launch_bounds__(TB) void node_items_kernel(const uint32_t* __restrict__ off,
                                                        const uint32_t* __restrict__ P, int64_t nn,
                                                        const int32_t* __restrict__ count,
                                                        uint32_t* __restrict__ nitems, uint32_t* __restrict__ prows) {
    const int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x;
    if (i < nn) leaf_items(P, off[i], off[i + 1], count[i], &nitems[i], &prows[i]);
}

// ---- work items ------------------------------------------------------------------
// One thread per item: its leaf is the last node whose first item is at or
// before it (nodes without items share their first-item index with the next
// node); it ends where the next item of the list starts.
__global__ __launch_bounds__(TB) void item_write_kernel(const uint32_t* __restrict__ P,
                                                        const uint32_t* __restrict__ l0,
                                                        const uint32_t* __restrict__ l1, int64_t nn,
                                                        const uint32_t* __restrict__ nitems,
                                                        const uint32_t* __restrict__ item0,
                                                        const uint32_t* __restrict__ n_items,
                                                        const uint32_t* __restrict__ pbase,
                                                        const int32_t* __restrict__ count,
                                                        int32_t* __restrict__ it_leaf, uint32_t* __restrict__ it_q0,
                                                        uint32_t* __restrict__ it_q1, uint32_t* __restrict__ it_pbase,
                                                        int32_t* __restrict__ leaf_item0,
                                                        int32_t* __restrict__ leaf_nitems,
                                                        int32_t* __restrict__ multi_leaf,
                                                        WalkTotals* __restrict__ res) {
    const uint32_t total = *n_items;
    // (gridDim.x * TB at most kListStep)
    for (uint32_t i = (uint32_t)(blockIdx.x * TB + threadIdx.x); i < total; i += gridDim.x * TB) {
        int64_t lo = 0, hi = nn - 1;
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) / 2;
            if (item0[mid] <= i) lo = mid;
            else hi = mid - 1;
        }
        const int64_t L = lo;
        const uint32_t n = nitems[L], k = i - item0[L];
        const uint32_t q0 = l0[L], q1 = l1[L];
        it_leaf[i] = (int32_t)L;
        it_q0[i] = item_start(P, q0, q1, k);
        it_q1[i] = k + 1u < n ? item_start(P, q0, q1, k + 1u) : q1;
        it_pbase[i] = n > 1u ? pbase[L] + k * (uint32_t)count[L] : 0u;
        if (k == 0u) {
            leaf_item0[L] = (int32_t)item0[L];
            leaf_nitems[L] = (int32_t)n;
            if (n > 1u) {
                multi_leaf[atomicAdd(&res->multi, 1u)] = (int32_t)L;
                atomicAdd(&res->rows, (unsigned long long)item_rows(n, count[L]));
            }
        }
    }
}

// The scans over the nodes, the items and the read-back of a small tree in one
// launch (the other form: a scan of two launches, the item kernel and the
// read-back's).
constexpr int kSmallNodes = 4096;
constexpr int SI = 1024;
__global__ __launch_bounds__(SI) void items_small_kernel(const uint32_t* __restrict__ P,
                                                         const uint32_t* __restrict__ l0,
                                                         const uint32_t* __restrict__ l1, int nn,
                                                         const uint32_t* __restrict__ nitems,
                                                         const uint32_t* __restrict__ prows,
                                                         const int32_t* __restrict__ count,
                                                         int32_t* __restrict__ it_leaf, uint32_t* __restrict__ it_q0,
                                                         uint32_t* __restrict__ it_q1,
                                                         uint32_t* __restrict__ it_pbase,
                                                         int32_t* __restrict__ leaf_item0,
                                                         int32_t* __restrict__ leaf_nitems,
                                                         int32_t* __restrict__ multi_leaf, WalkTotals* tot,
                                                         Mailbox mb) {
    constexpr int PER = kSmallNodes / SI;
    __shared__ uint32_t item0[kSmallNodes], pbase[kSmallNodes];
    __shared__ uint32_t wsum[SI / kWave];
    __shared__ uint32_t multi;
    __shared__ unsigned long long rows;
    const int tid = threadIdx.x;
    if (tid == 0) {
        multi = 0u;
        rows = 0ull;
    }
    uint32_t a[PER], p[PER], sa = 0u, sb = 0u;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = tid * PER + k;
        a[k] = i < nn ? nitems[i] : 0u;
        p[k] = i < nn ? prows[i] : 0u;
        sa += a[k];
        sb += p[k];
    }
    uint32_t n_items, n_rows;
    uint32_t ra = block_excl(sa, wsum, n_items);
    uint32_t rb = block_excl(sb, wsum, n_rows);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = tid * PER + k;
        item0[i] = ra;
        pbase[i] = rb;
        ra += a[k];
        rb += p[k];
    }
    __syncthreads();
    for (uint32_t i = tid; i < n_items; i += SI) {
        int lo = 0, hi = nn - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            if (item0[mid] <= i) lo = mid;
            else hi = mid - 1;
        }
        const uint32_t n = nitems[lo], k = i - item0[lo];
        const uint32_t q0 = l0[lo], q1 = l1[lo];
        it_leaf[i] = lo;
        it_q0[i] = item_start(P, q0, q1, k);
        it_q1[i] = k + 1u < n ? item_start(P, q0, q1, k + 1u) : q1;
        it_pbase[i] = n > 1u ? pbase[lo] + k * (uint32_t)count[lo] : 0u;
        if (k == 0u) {
            leaf_item0[lo] = (int32_t)item0[lo];
            leaf_nitems[lo] = (int32_t)n;
            if (n > 1u) {
                multi_leaf[atomicAdd(&multi, 1u)] = lo;
                atomicAdd(&rows, (unsigned long long)item_rows(n, count[lo]));
            }
        }
    }
    __syncthreads();
    if (tid == 0) {
        tot->multi = multi;
        tot->items = n_items;
        tot->partial = n_rows;
        tot->rows = rows;
    }
    __syncthreads();
    mailbox_write(mb, tot, (int)(offsetof(WalkTotals, scratch) / 4));
}

// Directed near particle interactions: sum over directed leaf pairs of
// n_t * n_s (self pairs n (n - 1)), a wavefront per target.
__global__ __launch_bounds__(TB) void near_work_kernel(const uint32_t* __restrict__ l0,
                                                       const uint32_t* __restrict__ l1,
                                                       const uint32_t* __restrict__ src, int64_t nn,
                                                       const int32_t* __restrict__ count,
                                                       unsigned long long* __restrict__ out) {
    const int lane = threadIdx.x & (kWave - 1);
    unsigned long long s = 0ull;
    for (int64_t i = (int64_t)blockIdx.x * (TB / kWave) + threadIdx.x / kWave; i < nn;
         i += (int64_t)gridDim.x * (TB / kWave)) {
        const unsigned long long na = (unsigned long long)count[i];
        for (uint32_t q = l0[i] + lane; q < l1[i]; q += kWave)
            s += (int64_t)src[q] == i ? na * (na - 1) : na * (unsigned long long)count[src[q]];
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
    if (lane == 0 && s) atomicAdd(out, s);
}

// Largest node count of the bucket route (1024 buckets of up to 512 targets).
constexpr int64_t kBucketNodes = (int64_t)1 << (kBucketBits + kLocalBits);

// Groups the directed entries of np pairs by target: lists [l0[t], l1[t]) of
// src.  part: the entries partitioned (scratch); scr: counts and starts.
template <typename Word, bool NEAR>
void bucket_lists(Tree& t, const DevBuf& pairs, int64_t np, DevBuf& part, DevBuf& scr, DevBuf& src, uint32_t* l0,
                  uint32_t* l1, const NearOut& no, WalkTotals* res, hipStream_t s) {
    Ctx* ctx = t.ctx;
    const int64_t nn = t.n_nodes, ne = 2 * np;
    const int all = bits_for(nn);
    const int hb = std::min(all, kBucketBits), lb = all - hb;
    const Split sp{NEAR ? 1 : 0, hb, lb};
    const int nb = NEAR ? 1 << hb : (int)(((nn - 1) >> lb) + 1);
    const int64_t tiles = std::max<int64_t>(1, cdiv(ne, PT));
    const int64_t rows = tiles <= kDirectRows ? tiles : cdiv(tiles, kRows);
    part.ensure(ctx, (size_t)std::max<int64_t>(ne, 1) * sizeof(Word));
    src.ensure(ctx, (size_t)std::max<int64_t>(ne, 1) * 4);
    scr.ensure(ctx, (size_t)((tiles + rows) * nb + NBK + 64) * 4);
    uint32_t* start = scr.as<uint32_t>();
    uint32_t* cnt = start + NBK + 64;
    const int2* pr = pairs.as<int2>();
    if (tiles == 1) {
        hipLaunchKernelGGL(bucket_scatter_kernel<Word>, dim3(1), dim3(PB), 0, s, pr, ne, sp, nb,
                           (const uint32_t*)nullptr, (const uint32_t*)nullptr, 1, part.as<Word>(), start, res);
        TFMM_LAUNCHED();
    } else {
        hipLaunchKernelGGL(bucket_count_kernel, dim3((unsigned)tiles), dim3(PB), 0, s, pr, ne, sp, nb, cnt);
        TFMM_LAUNCHED();
        uint32_t* M = cnt;
        if (tiles > kDirectRows) {
            M = cnt + tiles * nb;
            hipLaunchKernelGGL(bucket_rows_kernel, dim3((unsigned)rows, (unsigned)cdiv(nb, TB)), dim3(TB), 0, s, cnt,
                               tiles, nb, M);
            TFMM_LAUNCHED();
        }
        hipLaunchKernelGGL(bucket_starts_kernel, dim3(1), dim3(NBK), 0, s, M, rows, nb, start, res);
        TFMM_LAUNCHED();
        hipLaunchKernelGGL(bucket_scatter_kernel<Word>, dim3((unsigned)tiles), dim3(PB), 0, s, pr, ne, sp, nb,
                           (const uint32_t*)(tiles > kDirectRows ? cnt : nullptr), (const uint32_t*)M,
                           tiles > kDirectRows ? kRows : 1, part.as<Word>(), start, res);
        TFMM_LAUNCHED();
    }
    hipLaunchKernelGGL((bucket_lists_kernel<Word, NEAR>), dim3((unsigned)nb), dim3(LT), 0, s,
                       (const Word*)part.as<Word>(), (const uint32_t*)start, sp, nb, lb, nn, src.as<uint32_t>(), l0, l1,
                       no);
    TFMM_LAUNCHED();
}

// The same for larger trees: a stable sort by target of the directed entries
// (read straight from the pair array), then offsets from the sorted targets.
// With self_dummy, the second entry of a self pair gets key nn and sorts
// last, so the first off[nn] entries are the real ones; off[nn] is also
// written to *real_out if given.
void sorted_lists(Tree& t, const DevBuf& pairs, int64_t np, bool self_dummy, DevBuf& tgtbuf, DevBuf& src,
                  uint32_t* off, DevBuf& scr, DevBuf& scr2, uint32_t* real_out, hipStream_t s) {
    Ctx* ctx = t.ctx;
    const int64_t nn = t.n_nodes, ne = 2 * np;
    const int64_t room = std::max<int64_t>(ne, 1);
    tgtbuf.ensure(ctx, (size_t)room * 4);
    src.ensure(ctx, (size_t)room * 4);
    scr2.ensure(ctx, (size_t)room * 8 + 256);
    uint32_t* kalt = scr2.as<uint32_t>();
    int32_t* valt = reinterpret_cast<int32_t*>(kalt + room);
    const int bits = bits_for(self_dummy ? nn + 1 : nn);
    scr.ensure(ctx, sort_scratch_bytes(ne, sort_passes(bits)) + 1024);
    radix_sort_pairs(pairs.as<int2>(), np, self_dummy, (uint32_t)nn, tgtbuf.as<uint32_t>(), src.as<int32_t>(), kalt,
                     valt, bits, scr.p, ctx->dev_err, s);
    hipLaunchKernelGGL(csr_offsets_kernel, dim3(grid(cdiv(ne + 1, 4))), dim3(TB), 0, s,
                       (const uint32_t*)tgtbuf.as<uint32_t>(), ne, nn, off, real_out);
    TFMM_LAUNCHED();
}

}  // namespace

// Far lists on s: sources m2l_src[m2l_off[t]] .. [m2l_off[t + 1]].
void build_far_lists(Tree& t, hipStream_t s) {
    const int64_t nn = t.n_nodes;
    t.m2l_off.ensure(t.ctx, (size_t)(nn + 1) * 4);
    uint32_t* off = t.m2l_off.as<uint32_t>();
    if (nn <= 65536)
        bucket_lists<uint32_t, false>(t, t.m2l_pairs, t.n_m2l, t.scratch2, t.scratch, t.m2l_src, off, off + 1,
                                      NearOut{}, nullptr, s);
    else if (nn <= kBucketNodes)
        bucket_lists<uint64_t, false>(t, t.m2l_pairs, t.n_m2l, t.scratch2, t.scratch, t.m2l_src, off, off + 1,
                                      NearOut{}, nullptr, s);
    else
        sorted_lists(t, t.m2l_pairs, t.n_m2l, false, t.w_tg, t.m2l_src, off, t.scratch, t.scratch2, nullptr, s);
}

// Near lists (self pairs once) and their work items on s.  Every leaf has
// exactly one self pair, so the entry count is 2 n_near - n_leaves, which
// near_lists_end checks.
void build_near_lists(Tree& t, hipStream_t s) {
    Ctx* ctx = t.ctx;
    const int64_t nn = t.n_nodes, np = t.n_p2p, ne = 2 * np - t.n_leaves;
    t.w_res.ensure(ctx, sizeof(WalkTotals));
    WalkTotals* res = t.w_res.as<WalkTotals>();
    t.w_c.ensure(ctx, (size_t)std::max<int64_t>(2 * np, 1) * 4);
    uint32_t* P = t.w_c.as<uint32_t>();
    // list bounds: starts and ends, or nn + 1 offsets
    t.p2p_off.ensure(ctx, (size_t)(2 * nn + 1) * 4);
    uint32_t* l0 = t.p2p_off.as<uint32_t>();
    uint32_t* l1 = nn <= kBucketNodes ? l0 + nn : l0 + 1;
    t.p2p_l1 = l1;
    // per node: items and partial rows, and their offsets
    t.w_fl.ensure(ctx, (size_t)(nn + 1) * 16);
    uint32_t* nit = t.w_fl.as<uint32_t>();
    uint32_t* it0 = nit + (nn + 1);
    uint32_t* prw = it0 + (nn + 1);
    uint32_t* pbs = prw + (nn + 1);
    const NearOut no{t.nd_count.as<int32_t>(), P, nit, prw};
    if (nn <= 65536) {
        bucket_lists<uint32_t, true>(t, t.p2p_pairs, np, t.scratch2_b, t.scratch_b, t.p2p_src, l0, l1, no, res, s);
    } else if (nn <= kBucketNodes) {
        bucket_lists<uint64_t, true>(t, t.p2p_pairs, np, t.scratch2_b, t.scratch_b, t.p2p_src, l0, l1, no, res, s);
    } else {
        sorted_lists(t, t.p2p_pairs, np, true, t.w_tg_b, t.p2p_src, l0, t.scratch_b, t.scratch2_b,
                     &res->near_entries, s);
        t.scratch_b.ensure(ctx, scan_scratch_bytes(ne) + 256);
        exclusive_scan_gather_u32(t.p2p_src.as<int32_t>(), t.nd_count.as<int32_t>(), P, ne, t.scratch_b.p,
                                  res->scratch, s);
        hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(TB), 0, s, reinterpret_cast<int32_t*>(&res->multi),
                           (int64_t)1, 0);
        TFMM_LAUNCHED();
        hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(TB), 0, s, reinterpret_cast<int32_t*>(&res->rows),
                           (int64_t)2, 0);
        TFMM_LAUNCHED();
        hipLaunchKernelGGL(node_items_kernel, dim3(grid(nn)), dim3(TB), 0, s, (const uint32_t*)l0, (const uint32_t*)P,
                           nn, t.nd_count.as<int32_t>(), nit, prw);
        TFMM_LAUNCHED();
    }
    // a list has no more items than entries, so every item array is sized by ne
    const size_t ni = (size_t)std::max<int64_t>(ne, 1);
    t.it_leaf.ensure(ctx, ni * 4);
    t.it_q0.ensure(ctx, ni * 4);
    t.it_q1.ensure(ctx, ni * 4);
    t.it_pbase.ensure(ctx, ni * 4);
    t.leaf_item0.ensure(ctx, (size_t)(nn + 1) * 4);
    t.leaf_nitems.ensure(ctx, (size_t)(nn + 1) * 4);
    t.multi_leaf.ensure(ctx, (size_t)(nn + 1) * 4);
    t.multi_count = &res->multi;
    t.list_mb = 0u;
    if (nn <= kSmallNodes) {
        const Mailbox mb = mailbox_next(ctx);
        t.list_mb = mb.seq;
        hipLaunchKernelGGL(items_small_kernel, dim3(1), dim3(SI), 0, s, (const uint32_t*)P, (const uint32_t*)l0,
                           (const uint32_t*)l1, (int)nn, (const uint32_t*)nit, (const uint32_t*)prw,
                           t.nd_count.as<int32_t>(), t.it_leaf.as<int32_t>(), t.it_q0.as<uint32_t>(),
                           t.it_q1.as<uint32_t>(), t.it_pbase.as<uint32_t>(), t.leaf_item0.as<int32_t>(),
                           t.leaf_nitems.as<int32_t>(), t.multi_leaf.as<int32_t>(), res, mb);
        TFMM_LAUNCHED();
        return;
    }
    t.scratch_b.ensure(ctx, scan_scratch_bytes(nn) + 256);
    exclusive_scan2_u32(nit, it0, &res->items, prw, pbs, &res->partial, nn, t.scratch_b.p, s);
    hipLaunchKernelGGL(item_write_kernel, dim3((unsigned)std::min<int64_t>(2048, grid(ne))), dim3(TB), 0, s,
                       (const uint32_t*)P, (const uint32_t*)l0, (const uint32_t*)l1, nn, (const uint32_t*)nit,
                       (const uint32_t*)it0, (const uint32_t*)&res->items, (const uint32_t*)pbs,
                       t.nd_count.as<int32_t>(), t.it_leaf.as<int32_t>(), t.it_q0.as<uint32_t>(),
                       t.it_q1.as<uint32_t>(), t.it_pbase.as<uint32_t>(), t.leaf_item0.as<int32_t>(),
                       t.leaf_nitems.as<int32_t>(), t.multi_leaf.as<int32_t>(), res);
    TFMM_LAUNCHED();
}

// Reads the near lists' totals back.
void near_lists_end(Tree& t, hipStream_t s) {
    const int64_t ne = 2 * t.n_p2p - t.n_leaves;
    WalkTotals h;
    const uint32_t seq = t.list_mb;
    t.list_mb = 0u;
    if (seq) mailbox_wait(t.ctx, seq, offsetof(WalkTotals, scratch), &h, true, s);
    else read_back_bytes(t.ctx, t.w_res.p, offsetof(WalkTotals, scratch), &h, true, s);
    if ((int64_t)h.near_entries != ne)
        fail(TFMM_EDEVICE, "walk: near entry count " + std::to_string(h.near_entries) + " differs from " +
                               std::to_string(ne));
    if (!rows_fit(h.rows))
        fail(TFMM_ENOMEM, "near field: " + std::to_string(h.rows) + " partial sums exceed 2^32 - 1");
    t.n_near_int = -1;  // counted on request (near_interactions)
    t.n_items = h.items;
    t.n_partial = h.partial;
}

// Directed near particle interactions of the last walk (throughput
// accounting): one pass over the near lists, on the null stream after the
// device is idle, counted once per walk.
int64_t near_interactions(Tree& t) {
    if (!t.walk_valid) return -1;
    if (t.n_near_int >= 0) return t.n_near_int;
    TFMM_HIP(hipDeviceSynchronize());
    unsigned long long* acc = &t.w_res.as<WalkTotals>()->near_int;
    hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(TB), 0, nullptr, reinterpret_cast<int32_t*>(acc), (int64_t)2, 0);
    TFMM_LAUNCHED();
    const unsigned nb = (unsigned)std::min<int64_t>(1024, std::max<int64_t>(1, cdiv(t.n_nodes, TB / kWave)));
    hipLaunchKernelGGL(near_work_kernel, dim3(nb), dim3(TB), 0, nullptr, (const uint32_t*)t.p2p_off.as<uint32_t>(),
                       (const uint32_t*)t.p2p_l1, (const uint32_t*)t.p2p_src.as<uint32_t>(), t.n_nodes,
                       t.nd_count.as<int32_t>(), acc);
    TFMM_LAUNCHED();
    t.n_near_int = (int64_t)read_back(t.ctx, (const unsigned long long*)acc, nullptr);
    return t.n_near_int;
}

}  // namespace tfmm
