// Stable LSD radix sort of (key, int32 value) pairs, 8-bit digits.  After the
// key's digits, the particle sort of a forest takes the digits of the set that
// the value (a particle's input index) belongs to.
//
// One histogram kernel, or the caller's own, counts the digits of every pass at
// once (the global digit totals do not depend on the order of the keys).  Each pass is then a
// single kernel over 4096-key tiles: a tile scans the pass's digit totals
// itself (the output start of every digit), ranks its keys (wave ballots find
// the lanes sharing a digit, a per-wave LDS counter carries ranks across
// rounds), publishes its per-digit counts, and finds the number of keys with
// the same digit in all earlier tiles by looking back over their published
// counts (decoupled look-back: a tile publishes its own count before it
// waits, and earlier tiles publish running totals, so the look-back usually
// stops after a tile or two).  Tiles take their index from an atomic ticket,
// so a tile only ever waits for tiles that are already running.  A status word
// carries its own value, so relaxed device-scope atomics suffice.  The tile is
// staged in LDS in digit order and written out in contiguous runs.  Tile
// order = input order, so equal keys keep their input order (stable).
//
// Every wait is bounded: a look-back that spins past kSpinLimit polls sets a
// device error word, which the host checks at its next read-back; the kernel
// always runs to its end.
//
// The first pass (and the histogram) reads its input through a source: plain
// key and value arrays, or an array of node pairs read as directed entries
// (entry 2i = (x_i <- y_i), entry 2i + 1 = (y_i <- x_i)), which spares the
// lists an expansion pass before the sort.
#include <algorithm>

#include "common.h"

namespace tfmm {
namespace {

constexpr int RADIX = 256;
constexpr int kLookBack = 4;      // earlier tiles read per look-back step
constexpr int RB = 256;           // threads per block of the histogram (one digit per thread)
constexpr int MAXP = 10;         // passes of a 64-bit key and a set number
constexpr int kHistBlocks = 1024;
constexpr int kHistKeysPerThread = 16;  // fewer blocks, fewer global atomics
constexpr uint32_t kSpinLimit = 1u << 20;
// A pass: a tile's 4096 keys are ranked by 16 wavefronts, four keys per lane.
// Up to 2^20 keys a tile runs alone on its compute unit and its serial parts set
// the pace: the ranking rounds (with four wavefronts, 16 keys per lane, eight
// passes over 100000 keys took 94 us, over 2^18 111, over 2^20 177; now 76, 90,
// 153) and the look-back, where reading fewer and smaller words counts more
// than taking fewer steps (four words a step 153 us on 2^20 keys, eight 154, 16
// 164, 32 178).  Tiles of 2048 keys halve the ranking but double the look-back:
// 71 us on 100000 keys, 94 on 2^18, 196 on 2^20; of 8192 keys 97, 109 and 157.
// Splitting a pass into count, scan and scatter launches, without waits, is
// slower at every size: 234 against 153 us on 2^20 keys, 418 against 364 on
// 2^22 and 708 against 663 on 9e6 keys.
constexpr int kPassThreads = 1024;
constexpr int kPassKeys = 4;
constexpr int kPassTile = kPassThreads * kPassKeys;
// Tile status word: the two highest bits a flag (0 none, 1 own count, 2 running
// total including this tile), the others the value.  32 bits for sorts of fewer
// than 2^30 keys.
template <typename S>
struct Status {
    static constexpr int kBits = 8 * sizeof(S) - 2;
    static constexpr S kOwn = (S)1 << kBits, kTotal = (S)2 << kBits, kValue = ((S)1 << kBits) - 1;
};
constexpr int64_t kShortStatus = (int64_t)1 << 30;

__device__ __forceinline__ uint64_t lanemask_lt() {
    const int lane = threadIdx.x & (kWave - 1);
    return (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
}

// Lanes holding the same 8-bit digit (all 64 lanes must be active).
__device__ __forceinline__ uint64_t digit_peers(uint32_t d) { return same_lanes<8>(true, d); }

// Input sources.  load(i) gives entry i's key and value.
template <typename K>
struct ArraySrc {
    const K* k;
    const int32_t* v;
    __device__ __forceinline__ void load(int64_t i, K& key, int32_t& val) const {
        key = k[i];
        val = v[i];
    }
};

// Directed entries of node pairs.  With self_dummy set, the second entry of a
// pair (x, x) gets the key self_key (above every node id), so it sorts after
// all real entries.
struct PairSrc {
    const int2* p;
    uint32_t self_key;
    int self_dummy;
    __device__ __forceinline__ void load(int64_t i, uint32_t& key, int32_t& val) const {
        const int2 q = p[i >> 1];
        if (i & 1) {
            key = (self_dummy && q.x == q.y) ? self_key : (uint32_t)q.y;
            val = q.x;
        } else {
            key = (uint32_t)q.x;
            val = q.y;
        }
    }
};

// Digit of an entry.
struct KeyDigit {
    int shift;
    template <typename K>
    __device__ __forceinline__ uint32_t operator()(K key, int32_t) const {
        return (uint32_t)(key >> shift) & (RADIX - 1);
    }
};
struct SetDigit {
    const int64_t* off;
    int n_sets, shift;
    __device__ __forceinline__ uint32_t operator()(uint64_t, int32_t val) const {
        return (uint32_t)(set_of(off, n_sets, val) >> shift) & (RADIX - 1);
    }
};

__global__ __launch_bounds__(RB) void zero_u64_kernel(unsigned long long* __restrict__ p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * RB + threadIdx.x; i < n; i += (int64_t)gridDim.x * RB) p[i] = 0ull;
}

// Digit totals of every pass: LDS counters per block, then global atomics.
__global__ __launch_bounds__(RB) void radix_hist_pairs_kernel(PairSrc src, int64_t n, int passes,
                                                              uint32_t* __restrict__ ghist) {
    __shared__ uint32_t h[4][RADIX];
    for (int p = 0; p < 4; ++p) h[p][threadIdx.x] = 0u;
    __syncthreads();
    constexpr int U = kHistKeysPerThread;  // loads in flight per thread
    const int64_t stride = (int64_t)gridDim.x * RB * U;
    for (int64_t base = (int64_t)blockIdx.x * RB * U; base < n; base += stride) {
        uint32_t k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = base + (int64_t)u * RB + threadIdx.x;
            int32_t unused;
            k[u] = 0u;
            if (i < n) src.load(i, k[u], unused);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (base + (int64_t)u * RB + threadIdx.x < n) {
                for (int p = 0; p < passes; ++p)
                    atomicAdd(&h[p][(k[u] >> (8 * p)) & (RADIX - 1)], 1u);
            }
        }
    }
    __syncthreads();
    for (int p = 0; p < passes; ++p) {
        const uint32_t c = h[p][threadIdx.x];
        if (c) atomicAdd(&ghist[p * RADIX + threadIdx.x], c);
    }
}

template <typename K, typename S, typename Dig, typename Src>
__global__ __launch_bounds__(kPassThreads) void radix_pass_kernel(Src src, Dig digit, K* __restrict__ kout, int32_t* __restrict__ vout,
                                                        int64_t n,
                                                        const uint32_t* __restrict__ dcount,
                                                        S* __restrict__ status,
                                                        uint32_t* __restrict__ ticket, uint32_t* __restrict__ err) {
    using ST = Status<S>;
    constexpr int T = kPassThreads, RI = kPassKeys, RTILE = kPassTile, PW = T / kWave;
    static_assert(T >= RADIX, "a thread per digit");
    __shared__ uint16_t wcnt[PW][RADIX];
    __shared__ uint32_t dstart[RADIX];
    __shared__ S gbase[RADIX];
    __shared__ uint32_t wsum[RADIX / kWave];
    __shared__ uint32_t hsum[RADIX / kWave];
    __shared__ K skeys[RTILE];
    __shared__ int32_t svals[RTILE];
    __shared__ uint32_t s_tile;

    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    if (threadIdx.x == 0) s_tile = atomicAdd(ticket, 1u);
    const int d = threadIdx.x;
    const uint32_t hc = d < RADIX ? dcount[d] : 0u;  // all keys with this thread's digit
    for (int x = lane; x < RADIX; x += kWave) wcnt[w][x] = 0;
    __syncthreads();
    const int64_t tile = s_tile;

    const int64_t tile0 = tile * RTILE;
    const int64_t wbase = tile0 + (int64_t)w * (kWave * RI);
    K k[RI];
    int32_t v[RI];
    uint32_t rank[RI];
    uint32_t dig[RI];
#pragma unroll
    for (int r = 0; r < RI; ++r) {
        const int64_t i = wbase + (int64_t)r * kWave + lane;
        k[r] = (K)0;
        v[r] = 0;
        if (i < n) src.load(i, k[r], v[r]);
    }
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int r = 0; r < RI; ++r) {
        const int64_t i = wbase + (int64_t)r * kWave + lane;
        const bool valid = i < n;
        const uint32_t kd = valid ? digit(k[r], v[r]) : (uint32_t)RADIX - 1;
        dig[r] = kd;
        const uint64_t peers = digit_peers(kd);
        const uint32_t below = (uint32_t)__popcll(peers & lt);
        const uint32_t base = wcnt[w][kd];
        rank[r] = base + below;
        if (below == 0) wcnt[w][kd] = (uint16_t)(base + (uint32_t)__popcll(peers));
    }
    __syncthreads();

    const int64_t rem = n - tile0;
    const int valid_count = (int)(rem < RTILE ? rem : RTILE);
    uint32_t tot = 0, incl = 0, hincl = 0;
    S excl = 0;
    if (d < RADIX) {
        // per digit: exclusive offsets across waves and the tile's count
        for (int ww = 0; ww < PW; ++ww) {
            const uint32_t c = wcnt[ww][d];
            wcnt[ww][d] = (uint16_t)tot;
            tot += c;
        }
        // padding keys of the last tile were counted under digit 255: drop them
        const uint32_t real = (d == RADIX - 1) ? tot - (uint32_t)(RTILE - valid_count) : tot;

        // publish, look back over earlier tiles, publish the running total
        S* st = status + tile * RADIX;
        if (tile == 0) {
            __hip_atomic_store(&st[d], ST::kTotal | (S)real, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        } else {
            __hip_atomic_store(&st[d], ST::kOwn | (S)real, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // earlier tiles' words for this digit, kLook at a time (independent loads)
            constexpr int kLook = kLookBack;
            uint32_t spins = 0;
            int64_t j = tile - 1;
            bool done = false;
            while (!done && j >= 0) {
                S y[kLook];
#pragma unroll
                for (int b = 0; b < kLook; ++b)
                    y[b] = (j - b >= 0) ? __hip_atomic_load(&status[(j - b) * RADIX + d], __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT)
                                        : ST::kTotal;
                bool stalled = false;
#pragma unroll
                for (int b = 0; b < kLook; ++b) {
                    if (done || stalled) continue;
                    const S flag = y[b] & ~ST::kValue;
                    if (flag == 0) {
                        stalled = true;  // reload from tile j
                    } else {
                        excl += y[b] & ST::kValue;
                        --j;
                        if (flag == ST::kTotal) done = true;
                    }
                }
                if (stalled) {
                    if (++spins > kSpinLimit) {
                        atomicOr(err, 1u);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            __hip_atomic_store(&st[d], ST::kTotal | (excl + real), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // digit starts inside the tile and in the output (scans over digits)
        incl = tot;
        hincl = hc;
#pragma unroll
        for (int s = 1; s < kWave; s <<= 1) {
            const uint32_t u = __shfl_up(incl, s, kWave);
            const uint32_t hu = __shfl_up(hincl, s, kWave);
            if (lane >= s) {
                incl += u;
                hincl += hu;
            }
        }
        if (lane == kWave - 1) {
            wsum[w] = incl;
            hsum[w] = hincl;
        }
    }
    __syncthreads();
    if (d < RADIX) {
        uint32_t woff = 0, hoff = 0;
        for (int ww = 0; ww < w; ++ww) {
            woff += wsum[ww];
            hoff += hsum[ww];
        }
        dstart[d] = woff + incl - tot;
        gbase[d] = (S)(hoff + hincl - hc) + excl;
    }
    __syncthreads();

#pragma unroll
    for (int r = 0; r < RI; ++r) {
        const uint32_t pos = dstart[dig[r]] + wcnt[w][dig[r]] + rank[r];
        skeys[pos] = k[r];
        svals[pos] = v[r];
    }
    __syncthreads();

    for (int i = threadIdx.x; i < valid_count; i += T) {
        const K kk = skeys[i];
        const int32_t vv = svals[i];
        const uint32_t dd = digit(kk, vv);
        const int64_t dst = (int64_t)gbase[dd] + (i - (int64_t)dstart[dd]);
        kout[dst] = kk;
        vout[dst] = vv;
    }
}

// Scratch layout: digit counts [MAXP][RADIX] u32, tickets [MAXP] u32 (padded),
// then the tile status words [passes][tiles][RADIX], u32 or u64.
struct SortScratch {
    uint32_t* dcount;
    uint32_t* ticket;
    void* status;
    int64_t zero_words;  // u64 words to clear from the start of the scratch
};

SortScratch carve(void* scratch, int64_t n, int passes) {
    const int64_t nb = cdiv(n > 0 ? n : 1, kPassTile);
    auto* base = static_cast<unsigned long long*>(scratch);
    SortScratch s;
    s.dcount = reinterpret_cast<uint32_t*>(base);                          // MAXP*RADIX u32
    s.ticket = reinterpret_cast<uint32_t*>(base + MAXP * RADIX / 2);      // 64 u64 of room
    s.status = base + MAXP * RADIX / 2 + 64;
    s.zero_words = MAXP * RADIX / 2 + 64 + (int64_t)passes * nb * RADIX / (n < kShortStatus ? 2 : 1);
    return s;
}

// The passes of a sort of n entries read from src (scratch cleared, digit totals
// in place): the key's first bits, then the number of the value's set if off is
// given.  Pass ps writes (kout, vout) when the number of passes after it is
// even, else the alternate arrays, so the last pass always lands in (kout, vout).
template <typename K, typename Src>
void radix_passes(Src src, K* kout, int32_t* vout, K* kalt, int32_t* valt, int64_t n, int key_passes, int passes,
                  const int64_t* off, int n_sets, void* scratch, uint32_t* err, hipStream_t s) {
    const int64_t pt = cdiv(n, kPassTile);
    const SortScratch sc = carve(scratch, n, passes);
    for (int ps = 0; ps < passes; ++ps) {
        const bool to_out = ((passes - 1 - ps) & 1) == 0;
        K* ko = to_out ? kout : kalt;
        int32_t* vo = to_out ? vout : valt;
        const uint32_t* db = sc.dcount + ps * RADIX;
        auto pass = [&](auto word, auto from, auto digit) {
            using S = decltype(word);
            hipLaunchKernelGGL((radix_pass_kernel<K, S, decltype(digit), decltype(from)>), dim3((unsigned)pt),
                               dim3(kPassThreads), 0, s, from, digit, ko, vo, n, db,
                               static_cast<S*>(sc.status) + (int64_t)ps * pt * RADIX, sc.ticket + ps, err);
            TFMM_LAUNCHED();
        };
        auto sized = [&](auto from, auto digit) {
            // particles are always fewer
            if constexpr (sizeof(K) == 8) pass(uint32_t{}, from, digit);
            else if (n < kShortStatus) pass(uint32_t{}, from, digit);
            else pass((unsigned long long)0, from, digit);
        };
        // a later pass reads what the one before wrote, the other pair of arrays
        const ArraySrc<K> prev{to_out ? kalt : kout, to_out ? valt : vout};
        if (ps == 0) sized(src, KeyDigit{0});
        else if (ps < key_passes) sized(prev, KeyDigit{8 * ps});
        else if constexpr (sizeof(K) == 8) sized(prev, SetDigit{off, n_sets, 8 * (ps - key_passes)});
    }
}

}  // namespace

uint32_t* sort_counts(void* scratch, int64_t n, int passes, int64_t* clear_words) {
    const SortScratch sc = carve(scratch, n, passes);
    *clear_words = sc.zero_words;
    return sc.dcount;
}

void sort_clear(void* scratch, int64_t words, hipStream_t s) {
    hipLaunchKernelGGL(zero_u64_kernel, dim3((unsigned)std::min<int64_t>(2048, cdiv(words, RB))), dim3(RB), 0, s,
                       static_cast<unsigned long long*>(scratch), words);
    TFMM_LAUNCHED();
}

void radix_sort_particles(uint64_t* keys, int32_t* vals, uint64_t* keys_alt, int32_t* vals_alt, int64_t n,
                          const int64_t* off, int n_sets, void* scratch, uint32_t* err, hipStream_t s) {
    const int passes = kKeyPasses + set_passes(n_sets);
    const bool odd = passes & 1;
    radix_passes<uint64_t>(ArraySrc<uint64_t>{odd ? keys_alt : keys, odd ? vals_alt : vals}, keys, vals, keys_alt,
                           vals_alt, n, kKeyPasses, passes, off, n_sets, scratch, err, s);
}

size_t sort_scratch_bytes(int64_t n, int passes) { return (size_t)carve(nullptr, n, passes).zero_words * 8 + 256; }

void radix_sort_pairs(const int2* pairs, int64_t np, bool self_dummy, uint32_t self_key, uint32_t* keys,
                      int32_t* vals, uint32_t* keys_alt, int32_t* vals_alt, int bits, void* scratch, uint32_t* err,
                      hipStream_t s) {
    const int64_t n = 2 * np;
    if (n <= 0) return;
    const int passes = sort_passes(bits);
    int64_t words = 0;
    uint32_t* counts = sort_counts(scratch, n, passes, &words);
    sort_clear(scratch, words, s);
    const PairSrc src{pairs, self_key, self_dummy ? 1 : 0};
    const unsigned hb = (unsigned)std::min<int64_t>(kHistBlocks, cdiv(n, RB * kHistKeysPerThread));
    hipLaunchKernelGGL(radix_hist_pairs_kernel, dim3(hb), dim3(RB), 0, s, src, n, passes, counts);
    TFMM_LAUNCHED();
    radix_passes<uint32_t>(src, keys, vals, keys_alt, vals_alt, n, passes, passes, nullptr, 1, scratch, err, s);
}

}  // namespace tfmm
