// Octree construction on the GPU.
//
// Every quantity that feeds the multipole acceptance criterion (keys, centres
// of mass, r_max) is computed in FP64 in one fixed operation order, without
// contraction, so the node table and the interaction lists are reproducible
// bit for bit:
//   keys   q_d = min(2^21 - 1, floor((X_d - lo_d) * scale)), 21 bits per axis
//          interleaved x, y, z from the most significant bit;
//   order  stable sort by key;
//   nodes  (level l, prefix = key >> 3(21 - l)), split while count > n_leaf
//          and l < 21, numbered level by level in Morton order;
//   M, S   leaf: left-to-right sums over its sorted particles of m and m X;
//          inner node: sums over its children in digit order; Z = S / M;
//   r_max  sqrt of the largest ((dx*dx + dy*dy) + dz*dz) over the node's
//          particles, d = X - Z (the r_max of Eq. mac_criterion).
#pragma clang fp contract(off)

#include <algorithm>
#include <cmath>

#include "common.h"

namespace tfmm {
namespace {

constexpr int TB = 256;
constexpr uint32_t QMAX = (1u << kLevels) - 1u;

// Also clears the digit totals of the sort (counts: words to clear, or 0).
__global__ __launch_bounds__(TB) void bbox_partial_kernel(const double* __restrict__ pos, int64_t n,
                                                          double* __restrict__ part,
                                                          unsigned long long* __restrict__ clear, int64_t words) {
    for (int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x; i < words; i += (int64_t)gridDim.x * TB) clear[i] = 0ull;
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    int bad = 0;
    for (int64_t a = (int64_t)blockIdx.x * TB + threadIdx.x; a < n; a += (int64_t)gridDim.x * TB) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double v = pos[3 * a + d];
            bad |= !isfinite(v);
            lo[d] = v < lo[d] ? v : lo[d];
            hi[d] = v > hi[d] ? v : hi[d];
        }
    }
    __shared__ double sh[6][TB];
    __shared__ int s_bad;
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    if (bad) s_bad = 1;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        sh[d][threadIdx.x] = lo[d];
        sh[3 + d][threadIdx.x] = hi[d];
    }
    __syncthreads();
    for (int s = TB / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const double a = sh[d][threadIdx.x + s], b = sh[3 + d][threadIdx.x + s];
                if (a < sh[d][threadIdx.x]) sh[d][threadIdx.x] = a;
                if (b > sh[3 + d][threadIdx.x]) sh[3 + d][threadIdx.x] = b;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x < 6) part[7 * blockIdx.x + threadIdx.x] = sh[threadIdx.x][0];
    if (threadIdx.x == 6) part[7 * blockIdx.x + 6] = s_bad ? 1.0 : 0.0;
}

// The cube of the keys: out[0..2] lo, [3..5] hi, [6] ext = the largest
// extent (1 if all extents are 0), [7] scale = 2^21 / ext, [8] 1 if any
// coordinate is not finite.  Exact FP64 operations, no contraction.
__device__ void write_cube(const double* lo, const double* hi, bool bad, double* __restrict__ out) {
    double ext = 0.0;
    for (int d = 0; d < 3; ++d) {
        out[d] = lo[d];
        out[3 + d] = hi[d];
        const double e = hi[d] - lo[d];
        if (e > ext) ext = e;
    }
    if (ext == 0.0) ext = 1.0;
    const double scale = 2097152.0 / ext;
    out[6] = ext;
    out[7] = scale;
    out[8] = (bad || !isfinite(ext) || !isfinite(scale)) ? 1.0 : 0.0;
}

// The cube from the nb partial boxes, by every block that needs it (the
// result lands in LDS; block 0 also writes it to out).
__device__ void cube_of_parts(const double* __restrict__ part, int nb, double* __restrict__ out, double* cube) {
    constexpr int NW = TB / kWave;
    __shared__ double sh[NW][6];
    __shared__ int s_bad;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    if (tid == 0) s_bad = 0;
    __syncthreads();
    double v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int b = tid; b < nb; b += TB) {
        if (part[7 * b + 6] != 0.0) s_bad = 1;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double lo = part[7 * b + d], hi = part[7 * b + 3 + d];
            v[d] = lo < v[d] ? lo : v[d];
            v[3 + d] = hi > v[3 + d] ? hi : v[3 + d];
        }
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double lo = __shfl_xor(v[d], o, kWave), hi = __shfl_xor(v[3 + d], o, kWave);
            v[d] = lo < v[d] ? lo : v[d];
            v[3 + d] = hi > v[3 + d] ? hi : v[3 + d];
        }
    }
    if (lane == 0)
        for (int d = 0; d < 6; ++d) sh[wv][d] = v[d];
    __syncthreads();
    if (tid == 0) {
        double lo[3], hi[3];
        for (int d = 0; d < 3; ++d) {
            lo[d] = sh[0][d];
            hi[d] = sh[0][3 + d];
            for (int w = 1; w < NW; ++w) {
                lo[d] = sh[w][d] < lo[d] ? sh[w][d] : lo[d];
                hi[d] = sh[w][3 + d] > hi[d] ? sh[w][3 + d] : hi[d];
            }
        }
        write_cube(lo, hi, s_bad != 0, cube);
        if (blockIdx.x == 0)
            for (int d = 0; d < 9; ++d) out[d] = cube[d];
    }
    __syncthreads();
}

// Doubles in the order of unsigned integers, above 0 (the cleared word).
__device__ __forceinline__ unsigned long long ordered(double x) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    return (u >> 63) ? ~u : (u | 1ull << 63);
}
__device__ __forceinline__ double from_ordered(unsigned long long u) {
    return __longlong_as_double((long long)((u >> 63) ? (u & ~(1ull << 63)) : ~u));
}

// The bounding boxes of the sets of a forest, box k in the cleared words
// boxes + 8 k: the largest inverse ordered word of a coordinate (its minimum)
// [0..2], the largest ordered word [3..5], not finite [6].  A wavefront takes
// 1024 consecutive particles, whatever the sets, so that a large set is spread
// as a single one is (a workgroup per set took 19 us for 16 sets of 8192).
constexpr int kBoxRun = 1024;
__global__ __launch_bounds__(TB) void bbox_sets_kernel(const double* __restrict__ pos, int64_t n,
                                                       const int64_t* __restrict__ off, int n_sets,
                                                       unsigned long long* __restrict__ boxes) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t w0 = ((int64_t)blockIdx.x * (TB / kWave) + threadIdx.x / kWave) * kBoxRun;
    const int64_t w1 = w0 + kBoxRun < n ? w0 + kBoxRun : n;
    if (w0 >= n) return;
    for (int k = set_of(off, n_sets, w0); k < n_sets && off[k] < w1; ++k) {
        const int64_t a0 = off[k] > w0 ? off[k] : w0, a1 = off[k + 1] < w1 ? off[k + 1] : w1;
        double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
        bool bad = false;
#pragma unroll 4
        for (int64_t a = a0 + lane; a < a1; a += kWave) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const double v = pos[3 * a + d];
                bad |= !isfinite(v);
                lo[d] = v < lo[d] ? v : lo[d];
                hi[d] = v > hi[d] ? v : hi[d];
            }
        }
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const double x = __shfl_xor(lo[d], o, kWave), y = __shfl_xor(hi[d], o, kWave);
                lo[d] = x < lo[d] ? x : lo[d];
                hi[d] = y > hi[d] ? y : hi[d];
            }
        }
        unsigned long long* box = boxes + 8 * (int64_t)k;
        if (__ballot(bad) != 0ull && lane == 6) atomicMax(&box[6], 1ull);
        if (lane < 3) atomicMax(&box[lane], ~ordered(lane == 0 ? lo[0] : (lane == 1 ? lo[1] : lo[2])));
        else if (lane < 6) atomicMax(&box[lane], ordered(lane == 3 ? hi[0] : (lane == 4 ? hi[1] : hi[2])));
    }
}

// The cube of a set from its box.
__device__ __forceinline__ void cube_of_box(const unsigned long long* __restrict__ box, double* cube) {
    double lo[3], hi[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lo[d] = from_ordered(~box[d]);
        hi[d] = from_ordered(box[3 + d]);
    }
    write_cube(lo, hi, box[6] != 0ull, cube);
}

__device__ __forceinline__ uint64_t spread3(uint32_t v) {
    uint64_t x = v & 0x1fffffull;
    x = (x | (x << 32)) & 0x1f00000000ffffull;
    x = (x | (x << 16)) & 0x1f0000ff0000ffull;
    x = (x | (x << 8)) & 0x100f00f00f00f00full;
    x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

// The key of position x in a cube.
__device__ __forceinline__ uint64_t morton_key(const double* __restrict__ x, const double* cube) {
    uint32_t q[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double f = floor((x[d] - cube[d]) * cube[7]);
        q[d] = (f >= (double)QMAX) ? QMAX : (uint32_t)f;
    }
    return (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
}

// Keys and input indices; a block takes per * TB consecutive particles.  part:
// the partial boxes of a single set; boxes: those of a forest's sets.  counts:
// the sort's digit totals, 256 per pass, of the keys (counted here while they are
// in registers) and of the set numbers.  With the set number as one more digit
// of the particle sort, 16 sets of 8192 are sorted in 12 launches; sorting by key
// and then by set, each with its own clearing and counting, took 17 and 45 us
// more of a 684 us evaluation.
__global__ __launch_bounds__(TB) void morton_kernel(const double* __restrict__ pos, int64_t n,
                                                    const double* __restrict__ part, int nparts,
                                                    const unsigned long long* __restrict__ boxes,
                                                    double* __restrict__ cubes,
                                                    const int64_t* __restrict__ set_off, int n_sets, int per,
                                                    uint64_t* __restrict__ keys, int32_t* __restrict__ idx,
                                                    uint32_t* __restrict__ counts) {
    __shared__ double cube0[9];
    __shared__ uint32_t h[kKeyPasses][256];
    static_assert(TB == 256, "a thread per digit");
    const int64_t a0 = (int64_t)blockIdx.x * per * TB + threadIdx.x;
    // the block's only set, or -1
    int mine = 0;
    if (n_sets <= 1) {
        cube_of_parts(part, nparts, cubes, cube0);
    } else {
        const int64_t b0 = (int64_t)blockIdx.x * per * TB, b1 = b0 + (int64_t)per * TB;
        mine = set_of(set_off, n_sets, b0);
        if (mine != set_of(set_off, n_sets, b1 < n ? b1 - 1 : n - 1)) mine = -1;
        if (mine >= 0 && threadIdx.x == 0) cube_of_box(boxes + 8 * (int64_t)mine, cube0);
        if (blockIdx.x == 0) {
            for (int k = threadIdx.x; k < n_sets; k += TB) {
                const uint32_t size = (uint32_t)(set_off[k + 1] - set_off[k]);
                atomicAdd(&counts[kKeyPasses * 256 + (k & 255)], size);
                if (n_sets > 256) atomicAdd(&counts[(kKeyPasses + 1) * 256 + (k >> 8)], size);
                double c[9];
                cube_of_box(boxes + 8 * (int64_t)k, c);
#pragma unroll
                for (int d = 0; d < 9; ++d) cubes[16 * (int64_t)k + d] = c[d];
            }
        }
    }
#pragma unroll
    for (int p = 0; p < kKeyPasses; ++p) h[p][threadIdx.x] = 0u;
    __syncthreads();
    for (int k = 0; k < per; ++k) {
        const int64_t a = a0 + (int64_t)k * TB;
        if (a >= n) break;
        uint64_t key;
        if (mine >= 0) {
            key = morton_key(pos + 3 * a, cube0);
        } else {
            double c[9];
            cube_of_box(boxes + 8 * (int64_t)set_of(set_off, n_sets, a), c);
            key = morton_key(pos + 3 * a, c);
        }
        keys[a] = key;
        idx[a] = (int32_t)a;
#pragma unroll
        for (int p = 0; p < kKeyPasses; ++p) atomicAdd(&h[p][(uint32_t)(key >> (8 * p)) & 255u], 1u);
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < kKeyPasses; ++p) {
        const uint32_t c = h[p][threadIdx.x];
        if (c) atomicAdd(&counts[p * 256 + threadIdx.x], c);
    }
}

__device__ __forceinline__ double dist2(const double4& x, double cx, double cy, double cz) {
    const double dx = x.x - cx, dy = x.y - cy, dz = x.z - cz;
    return (dx * dx + dy * dy) + dz * dz;
}

// Maximum over each row of 16 lanes or over the wavefront, in every lane.
template <int LANES>
__device__ __forceinline__ double group_max(double v) {
    static_assert(LANES == 16 || LANES == kWave, "a row or a wavefront");
    auto up = [&](double u) { v = u > v ? u : v; };
    up(dpp<0xB1>(v));   // quad_perm [1,0,3,2]
    up(dpp<0x4E>(v));   // quad_perm [2,3,0,1]
    up(dpp<0x141>(v));  // row_half_mirror
    up(dpp<0x140>(v));  // row_mirror
    if (LANES == kWave) {
        up(__shfl_xor(v, 16, kWave));
        up(__shfl_xor(v, 32, kWave));
    }
    return v;
}

// A ball around one of the wavefront's particles (lane j of the first m lanes
// holds one) that holds them all.
__device__ __forceinline__ double4 ball_of(const double4& x, int m) {
    const int mid = m > kWave / 2 ? kWave / 2 : 0;
    const double cx = __shfl(x.x, mid, kWave), cy = __shfl(x.y, mid, kWave), cz = __shfl(x.z, mid, kWave);
    const double r2 = (int)(threadIdx.x & (kWave - 1)) < m ? dist2(x, cx, cy, cz) : 0.0;
    return make_double4(cx, cy, cz, sqrt(group_max<kWave>(r2)));
}

// Level at which a key boundary appears between two sorted neighbours (22 =
// equal keys, never a boundary).
__device__ __forceinline__ uint8_t boundary_level(uint64_t a, uint64_t b) {
    const uint64_t x = a ^ b;
    return x == 0 ? (uint8_t)(kLevels + 1) : (uint8_t)(kLevels - (63 - __clzll((long long)x)) / 3);
}

// A small single set in one workgroup: cube, keys, the whole stable sort (eight
// 8-bit passes in LDS, ranks by wavefront ballots as in the large sorts), the
// sorted particles and the boundary levels.  KPL keys per lane; keys past n
// are all ones and stay behind the last real key.  Replaces the cube, key,
// clearing, counting, eight pass and gather launches (14), each of which costs
// its launch and little else at these sizes: 31 us for a ball of 2048, where the
// launches took 80 us of kernels and as much again between them (step 330 -> 255
// us with the fewer launches of the rest of the build).
constexpr int ST = 1024;
constexpr int64_t kSmallSort = 8 * ST;
template <int KPL>
__global__ __launch_bounds__(ST) void small_sort_kernel(const double* __restrict__ pos,
                                                        const double* __restrict__ mass, int n,
                                                        double* __restrict__ cube_out, uint64_t* __restrict__ keys,
                                                        int32_t* __restrict__ perm, double4* __restrict__ Xm,
                                                        double4* __restrict__ balls, uint8_t* __restrict__ lvlb) {
    constexpr int NW = ST / kWave;
    __shared__ uint64_t sk[KPL * ST];
    __shared__ uint16_t sv[KPL * ST];
    __shared__ uint32_t wcnt[NW][256];
    __shared__ uint32_t dstart[256];
    __shared__ uint32_t wsum[4];
    __shared__ double box[NW][6];
    __shared__ double cube[9];
    __shared__ int s_bad;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int base = wv * (kWave * KPL) + lane;  // round r of this lane: base + r kWave
    if (tid == 0) s_bad = 0;
    __syncthreads();
    double v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    int bad = 0;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        const int a = base + r * kWave;
        if (a < n) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const double x = pos[3 * a + d];
                bad |= !isfinite(x);
                v[d] = x < v[d] ? x : v[d];
                v[3 + d] = x > v[3 + d] ? x : v[3 + d];
            }
        }
    }
    if (bad) s_bad = 1;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double lo = __shfl_xor(v[d], o, kWave), hi = __shfl_xor(v[3 + d], o, kWave);
            v[d] = lo < v[d] ? lo : v[d];
            v[3 + d] = hi > v[3 + d] ? hi : v[3 + d];
        }
    }
    if (lane == 0)
        for (int d = 0; d < 6; ++d) box[wv][d] = v[d];
    __syncthreads();
    if (tid == 0) {
        double lo[3], hi[3];
        for (int d = 0; d < 3; ++d) {
            lo[d] = box[0][d];
            hi[d] = box[0][3 + d];
            for (int w = 1; w < NW; ++w) {
                lo[d] = box[w][d] < lo[d] ? box[w][d] : lo[d];
                hi[d] = box[w][3 + d] > hi[d] ? box[w][3 + d] : hi[d];
            }
        }
        write_cube(lo, hi, s_bad != 0, cube);
        for (int d = 0; d < 9; ++d) cube_out[d] = cube[d];
    }
    __syncthreads();
    uint64_t k[KPL];
    uint16_t id[KPL];
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        const int a = base + r * kWave;
        id[r] = (uint16_t)a;
        k[r] = a < n ? morton_key(pos + 3 * a, cube) : ~0ull;
    }
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
    for (int pass = 0; pass < 8; ++pass) {
        const int shift = 8 * pass;
        for (int i = tid; i < NW * 256; i += ST) (&wcnt[0][0])[i] = 0u;
        __syncthreads();
        uint32_t rank[KPL];
#pragma unroll
        for (int r = 0; r < KPL; ++r) {
            const uint32_t d = (uint32_t)(k[r] >> shift) & 255u;
            const uint64_t peers = same_lanes<8>(true, d);
            const uint32_t below = (uint32_t)__popcll(peers & lt);
            const uint32_t first = wcnt[wv][d];
            rank[r] = first + below;
            if (below == 0) wcnt[wv][d] = first + (uint32_t)__popcll(peers);
        }
        __syncthreads();
        uint32_t tot = 0, incl = 0;
        if (tid < 256) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const uint32_t c = wcnt[w][tid];
                wcnt[w][tid] = tot;
                tot += c;
            }
            incl = tot;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const uint32_t u = (uint32_t)__shfl_up((int)incl, o, kWave);
                if (lane >= o) incl += u;
            }
            if (lane == kWave - 1) wsum[wv] = incl;
        }
        __syncthreads();
        if (tid < 256) {
            uint32_t off = 0;
            for (int w = 0; w < wv; ++w) off += wsum[w];
            dstart[tid] = off + incl - tot;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < KPL; ++r) {
            const uint32_t d = (uint32_t)(k[r] >> shift) & 255u;
            const uint32_t p = dstart[d] + wcnt[wv][d] + rank[r];
            sk[p] = k[r];
            sv[p] = id[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < KPL; ++r) {
            k[r] = sk[base + r * kWave];
            id[r] = sv[base + r * kWave];
        }
    }
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        const int j = base + r * kWave;
        double4 x = make_double4(0.0, 0.0, 0.0, 0.0);
        if (j < n) {
            const int a = id[r];
            keys[j] = k[r];
            perm[j] = a;
            x = make_double4(pos[3 * a], pos[3 * a + 1], pos[3 * a + 2], mass[a]);
            Xm[j] = x;
            lvlb[j] = j > 0 ? boundary_level(sk[j - 1], k[r]) : (uint8_t)0;
        }
        const int w0 = j - lane;
        if (w0 < n) {
            const double4 ball = ball_of(x, n - w0 < kWave ? n - w0 : kWave);
            if (lane == 0) balls[w0 / kWave] = ball;
        }
    }
}

// Sorted FP64 particles and the level at which a key boundary appears in front
// of each sorted position (22 = equal keys, never a boundary; 0 = the first
// particle of a set, where its root starts).  A wavefront's 64 particles also get
// a ball around one of them that holds them all (for r_max).
__global__ __launch_bounds__(TB) void gather_kernel(const double* __restrict__ pos,
                                                    const double* __restrict__ mass,
                                                    const uint64_t* __restrict__ keys,
                                                    const int32_t* __restrict__ perm, int64_t n,
                                                    const int64_t* __restrict__ set_off, int n_sets,
                                                    double4* __restrict__ Xm, double4* __restrict__ balls,
                                                    uint8_t* __restrict__ lvlb) {
    const int64_t j = (int64_t)blockIdx.x * TB + threadIdx.x;
    const int64_t w0 = j & ~(int64_t)(kWave - 1);
    if (w0 >= n) return;
    double4 x = make_double4(0.0, 0.0, 0.0, 0.0);
    if (j < n) {
        const int64_t a = perm[j];
        x = make_double4(pos[3 * a], pos[3 * a + 1], pos[3 * a + 2], mass[a]);
        Xm[j] = x;
    }
    const double4 ball = ball_of(x, n - w0 < kWave ? (int)(n - w0) : kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) balls[w0 / kWave] = ball;
    if (j >= n) return;
    uint8_t lb = 0;
    if (j > 0 && (n_sets <= 1 || set_off[set_of(set_off, n_sets, j)] != j)) lb = boundary_level(keys[j - 1], keys[j]);
    lvlb[j] = lb;
}

struct NodeArrays {
    int32_t* level;
    uint64_t* prefix;
    int32_t* first;
    int32_t* count;
    int32_t* child_first;
    int32_t* nchild;
    int32_t* parent;
};

// ---- octree from the sorted keys, all levels at once -------------------------
// With the split rule "count > n_leaf and level < 21", a particle's leaf level
// lambda(j) is one more than the deepest level at which its cell holds more
// than n_leaf particles (capped at 21; 0 when its whole set fits one leaf),
// and that happens exactly when some window of n_leaf + 1 consecutive sorted
// keys of its set around j shares the prefix of that level.  Position j then
// starts a node at every level l with lvlb[j] <= l <= lambda(j); the roots
// (level 0) start at the first particle of every set, so root k is node k.
// Node ids are level major and in position order inside a level, so an id is
// the level's first id plus the number of node starts at that level before j:
// per-level counts per block, scanned over blocks, plus wave ballots inside
// the block.
constexpr int NSLOT = kLevels + 2;  // levels 0..21 and a slot for the leaf count
constexpr int kMaxLeafWindow = 4096;

// Deepest level shared by keys[i] and keys[i + n_leaf] (21 if equal, -1 if the
// two belong to different sets).
__device__ __forceinline__ int8_t window_level(const uint64_t* __restrict__ keys, int64_t i, int n_leaf,
                                               const int64_t* __restrict__ set_off, int n_sets) {
    if (n_sets > 1 && set_off[set_of(set_off, n_sets, i) + 1] <= i + n_leaf) return (int8_t)-1;
    const uint64_t x = keys[i] ^ keys[i + n_leaf];
    return (x == 0) ? (int8_t)kLevels : (int8_t)(kLevels - (63 - __clzll((long long)x)) / 3 - 1);
}

// lambda(j) from the largest window level over the n_leaf + 1 windows that contain j
// (a sparse-table maximum in LDS), and per-level counts of node starts and of
// leaf starts for the block.
__global__ __launch_bounds__(TB) void leaf_level_kernel(const uint64_t* __restrict__ keys, int64_t n, int n_leaf,
                                                        const int64_t* __restrict__ set_off, int n_sets,
                                                        const uint8_t* __restrict__ lvlb, uint8_t* __restrict__ lam,
                                                        uint32_t* __restrict__ cnt, int64_t nblk,
                                                        uint32_t* __restrict__ done) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *done = 0u;
    constexpr int VMAX = (TB + kMaxLeafWindow + TB - 1) / TB;
    __shared__ int8_t m[TB + kMaxLeafWindow];
    __shared__ uint32_t wc[TB / kWave][NSLOT];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int64_t j0 = (int64_t)blockIdx.x * TB;
    const int64_t nw = n - n_leaf;
    const int TL = TB + n_leaf;
    for (int t = tid; t < TL; t += TB) {
        const int64_t i = j0 - n_leaf + t;
        m[t] = (i >= 0 && i < nw) ? window_level(keys, i, n_leaf, set_off, n_sets) : (int8_t)-1;
    }
    __syncthreads();
    const int w = n_leaf + 1;
    int span = 1;
    while (2 * span <= w) {
        int8_t v[VMAX];
#pragma unroll
        for (int q = 0; q < VMAX; ++q) {
            const int t = tid + q * TB;
            if (t < TL) {
                const int8_t x = m[t], y = (t + span < TL) ? m[t + span] : (int8_t)-1;
                v[q] = x > y ? x : y;
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < VMAX; ++q) {
            const int t = tid + q * TB;
            if (t < TL) m[t] = v[q];
        }
        __syncthreads();
        span *= 2;
    }
    const int64_t j = j0 + tid;
    const bool valid = j < n;
    int a = 99, b = 0;
    if (valid) {
        // windows [tid, tid + w) of the tile; m[t] covers [t, t + span)
        const int8_t x = m[tid], y = m[tid + w - span];
        const int bd = x > y ? x : y;
        b = bd < 0 ? 0 : (bd + 1 < kLevels ? bd + 1 : kLevels);
        lam[j] = (uint8_t)b;
        a = lvlb[j];
    }
    for (int l = 0; l <= kLevels; ++l) {
        const unsigned long long bl = __ballot(a <= l && l <= b);
        if (lane == 0) wc[wv][l] = (uint32_t)__popcll(bl);
    }
    const unsigned long long leaf = __ballot(a <= b);
    if (lane == 0) wc[wv][NSLOT - 1] = (uint32_t)__popcll(leaf);
    __syncthreads();
    if (tid < NSLOT) {
        uint32_t c = 0;
#pragma unroll
        for (int q = 0; q < TB / kWave; ++q) c += wc[q][tid];
        cnt[(int64_t)tid * nblk + blockIdx.x] = c;
    }
}

// Level boundaries and sizes of the octree (read back by the host once).
struct TreeHeader {
    int64_t LB[kLevels + 2];  // first node id of levels 0..21, then the node count
    int64_t max_level, n_nodes, n_leaves;
    int64_t nonfinite;        // a coordinate was not finite
};

// Exclusive scan over the blocks of one slot's counts (one block per slot):
// every thread takes a contiguous run of the counts, the run totals are
// scanned across the block (wave scans, then the waves' totals), and each
// thread writes its run's exclusive prefixes.  The block that finishes last
// (done: a counter that starts at zero) writes the header and the mailbox.
__global__ __launch_bounds__(TB) void slot_scan_kernel(uint32_t* __restrict__ cnt, int64_t nblk, uint32_t* tot,
                                                       uint32_t* done, const double* __restrict__ cubes, int n_sets,
                                                       TreeHeader* __restrict__ h, Mailbox mb) {
    __shared__ uint32_t wsum[TB / kWave];
    __shared__ int s_last;
    __shared__ int s_bad;
    uint32_t* c = cnt + (int64_t)blockIdx.x * nblk;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int64_t per = (nblk + TB - 1) / TB;
    const int64_t i0 = (int64_t)tid * per;
    const int64_t i1 = i0 + per < nblk ? i0 + per : nblk;
    uint32_t run = 0;
    for (int64_t i = i0; i < i1; ++i) run += c[i];
    uint32_t v = run;  // inclusive scan of the run totals over the wave
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t u = (uint32_t)__shfl_up((int)v, d, kWave);
        if (lane >= d) v += u;
    }
    if (lane == kWave - 1) wsum[wv] = v;
    if (tid == 0) s_bad = 0;
    __syncthreads();
    uint32_t base = 0, all = 0;
#pragma unroll
    for (int q = 0; q < TB / kWave; ++q) {
        if (q < wv) base += wsum[q];
        all += wsum[q];
    }
    uint32_t acc = base + v - run;
    for (int64_t i = i0; i < i1; ++i) {
        const uint32_t x = c[i];
        c[i] = acc;
        acc += x;
    }
    if (tid == 0) {
        __hip_atomic_store(&tot[blockIdx.x], all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t before = __hip_atomic_fetch_add(done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        s_last = before == gridDim.x - 1u;
    }
    __syncthreads();
    if (!s_last) return;
    for (int k = tid; k < n_sets; k += TB)
        if (cubes[16 * k + 8] != 0.0) s_bad = 1;
    __syncthreads();
    if (tid == 0) {
        h->nonfinite = s_bad;
        int64_t lb = 0, ml = 0;
        h->LB[0] = 0;
        for (int l = 0; l <= kLevels; ++l) {
            const uint32_t x = __hip_atomic_load(&tot[l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            lb += x;
            h->LB[l + 1] = lb;
            if (x > 0) ml = l;
        }
        h->max_level = ml;
        h->n_nodes = lb;
        h->n_leaves = (int64_t)__hip_atomic_load(&tot[NSLOT - 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    mailbox_write(mb, h, (int)(sizeof(TreeHeader) / 4));
}

__global__ __launch_bounds__(TB) void node_create_kernel(NodeArrays nd, int64_t n, const uint64_t* __restrict__ keys,
                                                         const uint8_t* __restrict__ lvlb,
                                                         const uint8_t* __restrict__ lam,
                                                         const uint32_t* __restrict__ boff, int64_t nblk,
                                                         const TreeHeader* __restrict__ h,
                                                         int32_t* __restrict__ leaf_of,
                                                         int32_t* __restrict__ leaves,
                                                         uint32_t* __restrict__ n_items) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_items = 0u;
    __shared__ unsigned long long bal[TB / kWave][NSLOT];
    __shared__ uint32_t woff[TB / kWave][NSLOT];
    __shared__ int64_t sLB[kLevels + 2];
    __shared__ uint32_t sboff[NSLOT];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int64_t j = (int64_t)blockIdx.x * TB + tid;
    const bool valid = j < n;
    const int a = valid ? (int)lvlb[j] : 99;
    const int b = valid ? (int)lam[j] : 0;
    for (int l = 0; l <= kLevels; ++l) {
        const unsigned long long bl = __ballot(a <= l && l <= b);
        if (lane == 0) bal[wv][l] = bl;
    }
    {
        const unsigned long long bl = __ballot(a <= b);  // a leaf starts here (at level b)
        if (lane == 0) bal[wv][NSLOT - 1] = bl;
    }
    if (tid < kLevels + 2) sLB[tid] = h->LB[tid];
    if (tid < NSLOT) sboff[tid] = boff[(int64_t)tid * nblk + blockIdx.x];
    __syncthreads();
    if (tid < NSLOT) {
        uint32_t run = 0;
#pragma unroll
        for (int q = 0; q < TB / kWave; ++q) {
            woff[q][tid] = run;
            run += (uint32_t)__popcll(bal[q][tid]);
        }
    }
    __syncthreads();
    if (!valid) return;
    const unsigned long long lt = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
    auto rank = [&](int l) -> int64_t {
        return (int64_t)sboff[l] + woff[wv][l] + (uint32_t)__popcll(bal[wv][l] & lt);
    };
    auto incl = [&](int l) -> int64_t { return rank(l) + ((a <= l && l <= b) ? 1 : 0); };
    leaf_of[j] = (int32_t)(sLB[b] + incl(b) - 1);
    // the list of leaves, in particle order (every user takes each leaf on its own)
    if (a <= b) leaves[rank(NSLOT - 1)] = (int32_t)(sLB[b] + rank(b));
    for (int l = a; l <= b; ++l) {
        const int64_t id = sLB[l] + rank(l);
        nd.level[id] = l;
        nd.prefix[id] = keys[j] >> (3 * (kLevels - l));
        nd.first[id] = (int32_t)j;
        nd.count[id] = 0;
        nd.nchild[id] = 0;
        nd.parent[id] = (l == 0) ? -1 : (int32_t)(sLB[l - 1] + incl(l - 1) - 1);
        nd.child_first[id] = (l + 1 <= b) ? (int32_t)(sLB[l + 1] + rank(l + 1)) : -1;
    }
}

// Particle counts (a node ends where the next node of its level starts if
// that node has the same parent, else where its parent ends; the roots,
// parent -1, end where the next root starts) and child counts (written by the
// last child).
__device__ __forceinline__ void node_finish(NodeArrays nd, int64_t c, int64_t n, const TreeHeader* __restrict__ h) {
    const int l = nd.level[c];
    const int32_t P = nd.parent[c];
    int64_t x = c, end = n;
    for (int lx = l; lx >= 0; --lx) {
        const int64_t nx = x + 1;
        if (nx < h->LB[lx + 1] && nd.parent[nx] == nd.parent[x]) {
            end = nd.first[nx];
            break;
        }
        x = nd.parent[x];
    }
    nd.count[c] = (int32_t)(end - nd.first[c]);
    if (P >= 0 && (c + 1 >= h->LB[l + 1] || nd.parent[c + 1] != P))
        nd.nchild[P] = (int32_t)(c - nd.child_first[P] + 1);
}

// Mass and centre of mass of leaf l of the list (a leaf ends where the next
// one starts: the list is in particle order).
__device__ __forceinline__ void geometry_leaf(const int32_t* __restrict__ leaves, int64_t l, int64_t n_leaves,
                                              const int32_t* __restrict__ first, int64_t n,
                                              const double4* __restrict__ Xm, double4* __restrict__ S,
                                              double4* __restrict__ Z) {
    const int32_t i = leaves[l];
    double M = 0.0, sx = 0.0, sy = 0.0, sz = 0.0;
    // loads issued eight at a time, sums kept strictly left to right
    const int32_t s0 = first[i], s1 = l + 1 < n_leaves ? first[leaves[l + 1]] : (int32_t)n;
    for (int32_t q = s0; q < s1; q += 8) {
        double4 p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (q + u < s1) p[u] = Xm[q + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (q + u < s1) {
                M = M + p[u].w;
                sx = sx + p[u].w * p[u].x;
                sy = sy + p[u].w * p[u].y;
                sz = sz + p[u].w * p[u].z;
            }
        }
    }
    S[i] = make_double4(sx, sy, sz, M);
    Z[i] = make_double4(sx / M, sy / M, sz / M, M);
}

// The first gl blocks: leaf geometry; the others: particle and child counts.
__global__ __launch_bounds__(TB) void node_finish_kernel(NodeArrays nd, int64_t nn, int64_t n,
                                                         const TreeHeader* __restrict__ h,
                                                         const int32_t* __restrict__ leaves, int64_t n_leaves,
                                                         unsigned gl, const double4* __restrict__ Xm,
                                                         double4* __restrict__ S, double4* __restrict__ Z) {
    if (blockIdx.x < gl) {
        const int64_t l = (int64_t)blockIdx.x * TB + threadIdx.x;
        if (l < n_leaves) geometry_leaf(leaves, l, n_leaves, nd.first, n, Xm, S, Z);
    } else {
        const int64_t c = (int64_t)(blockIdx.x - gl) * TB + threadIdx.x;
        if (c < nn) node_finish(nd, c, n, h);
    }
}

// Inner node: sums over its children in digit order.
__device__ __forceinline__ void geometry_inner(int32_t i, const int32_t* __restrict__ child_first,
                                               const int32_t* __restrict__ nchild, double4* __restrict__ S,
                                               double4* __restrict__ Z) {
    const int32_t nc = nchild[i];
    if (nc == 0) return;  // a leaf: done by geometry_leaf
    double M = 0.0, sx = 0.0, sy = 0.0, sz = 0.0;
    const int32_t c0 = child_first[i];
    for (int32_t c = c0; c < c0 + nc; ++c) {
        const double4 q = S[c];
        M = M + q.w;
        sx = sx + q.x;
        sy = sy + q.y;
        sz = sz + q.z;
    }
    S[i] = make_double4(sx, sy, sz, M);
    Z[i] = make_double4(sx / M, sy / M, sz / M, M);
}

// Inner nodes of one level (the level below is done).
__global__ __launch_bounds__(TB) void geometry_level_kernel(const int32_t* __restrict__ child_first,
                                                            const int32_t* __restrict__ nchild, int32_t lb,
                                                            int32_t le, double4* __restrict__ S,
                                                            double4* __restrict__ Z) {
    const int32_t i = lb + blockIdx.x * TB + threadIdx.x;
    if (i < le) geometry_inner(i, child_first, nchild, S, Z);
}

// Inner nodes of the top levels 0..top in one block, deepest first.
struct LevelBounds {
    int32_t b[kLevels + 2];
};
__global__ __launch_bounds__(TB) void geometry_top_kernel(const int32_t* __restrict__ child_first,
                                                          const int32_t* __restrict__ nchild, LevelBounds lv, int top,
                                                          double4* __restrict__ S, double4* __restrict__ Z) {
    for (int L = top; L >= 0; --L) {
        for (int32_t i = lv.b[L] + (int32_t)threadIdx.x; i < lv.b[L + 1]; i += TB) geometry_inner(i, child_first, nchild, S, Z);
        __syncthreads();
    }
}

// Exact r_max, the maximum squared distance of a node's particles from its
// centre of mass, and the walk's packed record of the node: geo = (centre of
// mass, r_max), top = (child count + 16 x the siblings from this node to its
// last, level, first child, set).  A row of 16 lanes per node; nodes of more
// than kBallsFrom particles are listed (in any order) as items of up to RCH
// particles, which a wavefront each takes through the balls of the sorted
// particles.  The items of a node of more than RCH meet in an atomicMax on the
// bits of the non-negative double, and rmax_final_kernel finishes it.  Up to
// kWaveNodes particles a wavefront takes a node, whole, and that launch is all.
//
// Bound by latency, a node being a chain of dependent loads, and on 2^22
// particles by the reads.  With a wavefront for every node and all distances
// looked at, the three launches took 44 us on 100000 particles, 67 on 2^20 and
// 219 on 2^22; now 27, 47 and 120.  Items from 200 particles cost 27, 52 and 126
// us, from 800 27, 48 and 125; rows of 16 lanes for nodes of any size 64, 116
// and 157.
constexpr int RCH = 4096;          // particles of an item: one ball per lane
constexpr int kBallsFrom = 512;
constexpr int kWaveNodes = 4 * RCH;

struct NodePack {
    const int64_t* set_off;
    int n_sets;
    double* rmax;
    double4* geo;
    int4* top;
};

__device__ __forceinline__ void pack_node(const NodeArrays& nd, const NodePack& pk, int32_t i, const double4& z,
                                          double r2) {
    const double r = sqrt(r2);
    const int32_t P = nd.parent[i];
    const int sib = P < 0 ? 1 : (int)(nd.child_first[P] + nd.nchild[P] - i);
    pk.rmax[i] = r;
    pk.geo[i] = make_double4(z.x, z.y, z.z, r);
    pk.top[i] = make_int4(nd.nchild[i] | (sib << 4), nd.level[i], nd.child_first[i],
                          set_of(pk.set_off, pk.n_sets, nd.first[i]));
}

template <int LANES>
__device__ __forceinline__ double max_r2(const double4* __restrict__ Xm, int32_t s0, int32_t s1, const double4& z) {
    double m = 0.0;
#pragma unroll 4
    for (int32_t s = s0 + (int32_t)(threadIdx.x & (LANES - 1)); s < s1; s += LANES) {
        const double d2 = dist2(Xm[s], z.x, z.y, z.z);
        m = d2 > m ? d2 : m;
    }
    return group_max<LANES>(m);
}

// The same, best for up to some RCH particles, through the balls of the 64-particle groups:
// a group's distances are looked at only if its ball reaches beyond the largest
// of the farthest reaching group.  The factor and the last term cover the
// rounding of the bound (the term where squares underflow), so the maximum is
// exactly max_r2's.  best: a value known not to exceed it, or 0.
__device__ __forceinline__ double max_r2_balls(const double4* __restrict__ Xm, const double4* __restrict__ balls,
                                               int32_t s0, int32_t s1, const double4& z, double best) {
    constexpr int U = 4;  // groups in flight
    const int lane = threadIdx.x & (kWave - 1);
    auto group = [&](int32_t b) {
        const int32_t s = b * kWave + lane;
        return s >= s0 && s < s1 ? dist2(Xm[s], z.x, z.y, z.z) : 0.0;
    };
    const int32_t last = (s1 - 1) / kWave;
    for (int32_t b0 = s0 / kWave; b0 <= last; b0 += kWave) {
        double reach = -1.0;
        if (b0 + lane <= last) {
            const double4 c = balls[b0 + lane];
            const double u = sqrt(dist2(c, z.x, z.y, z.z)) + c.w;
            reach = u * u * (1.0 + 1e-12) + 1e-290;
        }
        const double top = group_max<kWave>(reach);
        if (!(top > best)) continue;
        const int k = __ffsll((unsigned long long)__ballot(reach == top)) - 1;
        const double m = group_max<kWave>(group(b0 + k));
        best = m > best ? m : best;
        uint64_t todo = __ballot(reach > best) & ~(1ull << k);
        double far = 0.0;
        while (todo != 0ull) {
            double d[U];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int g = todo != 0ull ? __ffsll((unsigned long long)todo) - 1 : k;
                todo &= todo - 1ull;
                d[q] = group(b0 + g);
            }
#pragma unroll
            for (int q = 0; q < U; ++q) far = d[q] > far ? d[q] : far;
        }
        far = group_max<kWave>(far);
        best = far > best ? far : best;
    }
    return best;
}

template <int LANES>
__global__ __launch_bounds__(TB) void rmax_kernel(NodeArrays nd, int64_t nn, const double4* __restrict__ Xm,
                                                  const double4* __restrict__ balls, const double4* __restrict__ Z,
                                                  NodePack pk,
                                                  unsigned long long* __restrict__ r2bits, int2* __restrict__ items,
                                                  uint32_t* __restrict__ n_items) {
    // room for the block's items in one step
    __shared__ uint32_t mine, at0;
    if (threadIdx.x == 0) mine = 0u;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * (TB / LANES) + threadIdx.x / LANES;
    const int lane = threadIdx.x & (LANES - 1);
    const int32_t s0 = i < nn ? nd.first[i] : 0, cnt = i < nn ? nd.count[i] : 0;
    const bool listed = LANES < kWave && cnt > kBallsFrom;
    const int nc = (cnt + RCH - 1) / RCH;
    uint32_t at = 0u;
    if (listed && lane == 0) {
        r2bits[i] = 0ull;
        at = atomicAdd(&mine, (uint32_t)nc);
    }
    __syncthreads();
    if (threadIdx.x == 0 && mine != 0u) at0 = atomicAdd(n_items, mine);
    __syncthreads();
    if (i >= nn) return;
    if (listed) {
        at = at0 + (uint32_t)__shfl((int)at, 0, LANES);
        for (int k = lane; k < nc; k += LANES) items[at + k] = make_int2((int32_t)i, k);
        return;
    }
    const double4 z = Z[i];
    const double m = LANES == kWave && cnt > kBallsFrom ? max_r2_balls(Xm, balls, s0, s0 + cnt, z, 0.0)
                                                        : max_r2<LANES>(Xm, s0, s0 + cnt, z);
    if (lane == 0) pack_node(nd, pk, (int32_t)i, z, m);
}
__global__ __launch_bounds__(TB) void rmax_items_kernel(const uint32_t* __restrict__ n_items,
                                                        const int2* __restrict__ items, NodeArrays nd,
                                                        const double4* __restrict__ Xm,
                                                        const double4* __restrict__ balls,
                                                        const double4* __restrict__ Z, NodePack pk,
                                                        unsigned long long* __restrict__ r2bits) {
    const uint32_t ni = *n_items;
    for (uint32_t q = blockIdx.x * (TB / kWave) + threadIdx.x / kWave; q < ni; q += gridDim.x * (TB / kWave)) {
        const int2 it = items[q];
        const int32_t i = it.x, cnt = nd.count[i];
        const int32_t s0 = nd.first[i] + it.y * RCH, e = nd.first[i] + cnt;
        const double4 z = Z[i];
        const bool whole = cnt <= RCH;
        const double best = whole ? 0.0
                                  : __longlong_as_double((long long)__hip_atomic_load(&r2bits[i], __ATOMIC_RELAXED,
                                                                                      __HIP_MEMORY_SCOPE_AGENT));
        const double m = max_r2_balls(Xm, balls, s0, s0 + RCH < e ? s0 + RCH : e, z, best);
        if ((threadIdx.x & (kWave - 1)) == 0) {
            if (whole) pack_node(nd, pk, i, z, m);
            else if (m > best) atomicMax(&r2bits[i], (unsigned long long)__double_as_longlong(m));
        }
    }
}
__global__ __launch_bounds__(TB) void rmax_final_kernel(const uint32_t* __restrict__ n_items,
                                                        const int2* __restrict__ items, NodeArrays nd,
                                                        const double4* __restrict__ Z, NodePack pk,
                                                        const unsigned long long* __restrict__ r2bits) {
    const uint32_t ni = *n_items;
    for (uint32_t k = blockIdx.x * TB + threadIdx.x; k < ni; k += gridDim.x * TB) {
        const int2 it = items[k];
        if (it.y == 0 && nd.count[it.x] > RCH) pack_node(nd, pk, it.x, Z[it.x], __longlong_as_double((long long)r2bits[it.x]));
    }
}

template <typename T>
__global__ __launch_bounds__(TB) void sources_kernel(const double4* __restrict__ Xm,
                                                     const int32_t* __restrict__ leaf_of,
                                                     const double4* __restrict__ Z, int64_t n,
                                                     typename Vec4<T>::type* __restrict__ out) {
    const int64_t j = (int64_t)blockIdx.x * TB + threadIdx.x;
    if (j >= n) return;
    const double4 x = Xm[j];
    const double4 z = Z[leaf_of[j]];
    typename Vec4<T>::type r;
    r.x = (T)(x.x - z.x);
    r.y = (T)(x.y - z.y);
    r.z = (T)(x.z - z.z);
    r.w = (T)x.w;
    out[j] = r;
}

unsigned grid(int64_t n) { return (unsigned)cdiv(n > 0 ? n : 1, TB); }

NodeArrays node_arrays(Tree& t) {
    return NodeArrays{t.nd_level.as<int32_t>(), t.nd_prefix.as<uint64_t>(), t.nd_first.as<int32_t>(),
                      t.nd_count.as<int32_t>(), t.nd_child_first.as<int32_t>(), t.nd_nchild.as<int32_t>(),
                      t.nd_parent.as<int32_t>()};
}

void ensure_nodes(Tree& t, int64_t cap, int64_t keep, hipStream_t s) {
    (void)keep;
    const size_t c = (size_t)cap;
    t.nd_level.ensure_keep(t.ctx, c * 4, s);
    t.nd_prefix.ensure_keep(t.ctx, c * 8, s);
    t.nd_first.ensure_keep(t.ctx, c * 4, s);
    t.nd_count.ensure_keep(t.ctx, c * 4, s);
    t.nd_child_first.ensure_keep(t.ctx, c * 4, s);
    t.nd_nchild.ensure_keep(t.ctx, c * 4, s);
    t.nd_parent.ensure_keep(t.ctx, c * 4, s);
}

}  // namespace

void upload(Tree& t, DevBuf& dst, const void* src, size_t bytes, int slot, hipStream_t s) {
    if (bytes > kStageSlot) fail(TFMM_EINVAL, "set table too large");
    if (!t.stage) {
        TFMM_HIP(hipHostMalloc(&t.stage, 2 * kStageSlot, hipHostMallocDefault));
        TFMM_HIP(hipEventCreateWithFlags(&t.stage_ev, hipEventDisableTiming));
    } else {
        // the previous copy out of the staging area has finished reading it
        TFMM_HIP(hipEventSynchronize(t.stage_ev));
    }
    char* h = static_cast<char*>(t.stage) + (size_t)slot * kStageSlot;
    std::memcpy(h, src, bytes);
    dst.ensure(t.ctx, bytes);
    TFMM_HIP(hipMemcpyAsync(dst.p, h, bytes, hipMemcpyHostToDevice, s));
    TFMM_HIP(hipEventRecord(t.stage_ev, s));
}

void build_tree(Tree& t, const double* pos, const double* mass, hipStream_t s) {
    Ctx* ctx = t.ctx;
    const int64_t n = t.n;
    const size_t un = (size_t)n;
    // what was derived from the particles before goes with them
    t.built = false;
    t.walk_valid = false;
    t.mom_p = -1;
    t.src_prec = -1;

    const int ns = t.n_sets;
    const int64_t* soff = ns > 1 ? t.set_off.as<int64_t>() : nullptr;
    const int64_t nblk = cdiv(n, TB);
    const int nbb = (int)std::min<int64_t>(256, nblk);
    const int passes = kKeyPasses + set_passes(ns);
    int64_t sort_words = 0;
    sort_counts(nullptr, n, passes, &sort_words);
    // the sort's scratch, then the boxes of a forest's sets
    const int64_t box_words = ns > 1 ? 8 * (int64_t)ns : 0;
    t.scratch.ensure(ctx, (size_t)(sort_words + box_words) * 8 + 512);
    // the key cubes, then the partial boxes of a single set
    t.cube.ensure(ctx, (size_t)(ns * 16 + nbb * 7) * sizeof(double));
    double* cube = t.cube.as<double>();
    double* part = cube + ns * 16;
    t.keys.ensure(ctx, un * 8);
    t.perm.ensure(ctx, un * 4);
    t.Xm.ensure(ctx, un * 32);
    t.lvlb.ensure(ctx, un);
    t.balls.ensure(ctx, (size_t)cdiv(n, kWave) * 32);
    t.owner.ensure(ctx, un);
    t.leaf_of.ensure(ctx, un * 4);
    // header, a counter of finished blocks, the count of r_max items
    t.scratch2.ensure(ctx, sizeof(TreeHeader) + 256);
    TreeHeader* hdr = t.scratch2.as<TreeHeader>();
    uint32_t* done = reinterpret_cast<uint32_t*>(hdr + 1);
    uint32_t* n_items = done + 1;
    uint8_t* lam = t.owner.as<uint8_t>();
    t.flags.ensure(ctx, (size_t)(NSLOT * nblk + NSLOT) * 4);
    uint32_t* cnt = t.flags.as<uint32_t>();
    uint32_t* tot = cnt + NSLOT * nblk;

    // cubes, keys, stable order (by set, then by key), sorted particles and
    // boundary levels, on the device (no read-back)
    if (ns == 1 && n <= kSmallSort) {
        auto run = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(1), dim3(ST), 0, s, pos, mass, (int)n, cube, t.keys.as<uint64_t>(),
                               t.perm.as<int32_t>(), t.Xm.as<double4>(), t.balls.as<double4>(),
                               t.lvlb.as<uint8_t>());
            TFMM_LAUNCHED();
        };
        switch (cdiv(n, ST)) {
            case 1: run(small_sort_kernel<1>); break;
            case 2: run(small_sort_kernel<2>); break;
            case 3: run(small_sort_kernel<3>); break;
            case 4: run(small_sort_kernel<4>); break;
            case 5: run(small_sort_kernel<5>); break;
            case 6: run(small_sort_kernel<6>); break;
            case 7: run(small_sort_kernel<7>); break;
            default: run(small_sort_kernel<8>);
        }
    } else {
        t.keys2.ensure(ctx, un * 8);
        t.perm2.ensure(ctx, un * 4);
        uint32_t* counts = sort_counts(t.scratch.p, n, passes, &sort_words);
        unsigned long long* boxes = t.scratch.as<unsigned long long>() + sort_words;
        if (ns > 1) {
            sort_clear(t.scratch.p, sort_words + box_words, s);
            hipLaunchKernelGGL(bbox_sets_kernel, dim3((unsigned)cdiv(n, (int64_t)kBoxRun * (TB / kWave))), dim3(TB), 0,
                               s, pos, n, soff, ns, boxes);
        } else {
            hipLaunchKernelGGL(bbox_partial_kernel, dim3(nbb), dim3(TB), 0, s, pos, n, part,
                               t.scratch.as<unsigned long long>(), sort_words);
        }
        TFMM_LAUNCHED();
        // blocks of 1024 particles, of 4096 when there are many (a block adds up
        // to 2048 digit totals); an odd number of sort passes starts from the
        // other arrays
        const int per = n < (1 << 19) ? 4 : 16;
        const bool odd = passes & 1;
        hipLaunchKernelGGL(morton_kernel, dim3((unsigned)cdiv(n, (int64_t)per * TB)), dim3(TB), 0, s, pos, n,
                           (const double*)part, nbb, (const unsigned long long*)boxes, cube, soff, ns, per,
                           (odd ? t.keys2 : t.keys).as<uint64_t>(), (odd ? t.perm2 : t.perm).as<int32_t>(), counts);
        TFMM_LAUNCHED();
        radix_sort_particles(t.keys.as<uint64_t>(), t.perm.as<int32_t>(), t.keys2.as<uint64_t>(),
                             t.perm2.as<int32_t>(), n, soff, ns, t.scratch.p, ctx->dev_err, s);
        hipLaunchKernelGGL(gather_kernel, dim3(grid(n)), dim3(TB), 0, s, pos, mass, t.keys.as<uint64_t>(),
                           t.perm.as<int32_t>(), n, soff, ns, t.Xm.as<double4>(), t.balls.as<double4>(),
                           t.lvlb.as<uint8_t>());
        TFMM_LAUNCHED();
    }

    // octree: leaf level of every particle, node starts per level, node table
    hipLaunchKernelGGL(leaf_level_kernel, dim3((unsigned)nblk), dim3(TB), 0, s,
                       (const uint64_t*)t.keys.as<uint64_t>(), n, t.n_leaf, soff, ns,
                       (const uint8_t*)t.lvlb.as<uint8_t>(), lam, cnt, nblk, done);
    TFMM_LAUNCHED();
    const Mailbox mb = mailbox_next(ctx);
    hipLaunchKernelGGL(slot_scan_kernel, dim3(NSLOT), dim3(TB), 0, s, cnt, nblk, tot, done, (const double*)cube, ns,
                       hdr, mb);
    TFMM_LAUNCHED();
    TreeHeader H;
    mailbox_wait(ctx, mb.seq, sizeof(TreeHeader), &H, true, s);
    if (H.nonfinite) fail(TFMM_EINVAL, "positions contain non-finite values");
    t.n_nodes = H.n_nodes;
    t.max_level = (int)H.max_level;
    t.n_leaves = H.n_leaves;
    t.level_begin.assign((size_t)t.max_level + 2, 0);
    for (int l = 0; l <= t.max_level + 1; ++l) t.level_begin[(size_t)l] = H.LB[l];
    const int64_t nn = t.n_nodes;
    ensure_nodes(t, std::max<int64_t>(nn, 1), 0, s);
    NodeArrays nd = node_arrays(t);
    t.leaves.ensure(ctx, (size_t)std::max<int64_t>(t.n_leaves, 1) * 4);
    t.nd_S.ensure(ctx, (size_t)nn * 32);
    t.nd_Z.ensure(ctx, (size_t)nn * 32);
    hipLaunchKernelGGL(node_create_kernel, dim3((unsigned)nblk), dim3(TB), 0, s, nd, n,
                       (const uint64_t*)t.keys.as<uint64_t>(), (const uint8_t*)t.lvlb.as<uint8_t>(),
                       (const uint8_t*)lam, (const uint32_t*)cnt, nblk, (const TreeHeader*)hdr,
                       t.leaf_of.as<int32_t>(), t.leaves.as<int32_t>(), n_items);
    TFMM_LAUNCHED();
    const unsigned gl = grid(t.n_leaves);
    hipLaunchKernelGGL(node_finish_kernel, dim3(gl + grid(nn)), dim3(TB), 0, s, nd, nn, n, (const TreeHeader*)hdr,
                       (const int32_t*)t.leaves.as<int32_t>(), t.n_leaves, gl, (const double4*)t.Xm.as<double4>(),
                       t.nd_S.as<double4>(), t.nd_Z.as<double4>());
    TFMM_LAUNCHED();

    // geometry of the inner nodes level by level, deepest first; the
    // top levels (at most kTopNodes nodes together) in a single block
    {
        constexpr int64_t kTopNodes = 1024;
        int top = -1;
        while (top + 1 <= t.max_level && t.level_begin[(size_t)top + 2] <= kTopNodes) ++top;
        for (int L = t.max_level - 1; L > top; --L) {
            const int32_t b = (int32_t)t.level_begin[L], e = (int32_t)t.level_begin[L + 1];
            if (e <= b) continue;
            hipLaunchKernelGGL(geometry_level_kernel, dim3(grid(e - b)), dim3(TB), 0, s, nd.child_first, nd.nchild,
                               b, e, t.nd_S.as<double4>(), t.nd_Z.as<double4>());
            TFMM_LAUNCHED();
        }
        if (top >= 0) {
            LevelBounds lv{};
            for (int L = 0; L <= top + 1; ++L) lv.b[L] = (int32_t)t.level_begin[L];
            hipLaunchKernelGGL(geometry_top_kernel, dim3(1), dim3(TB), 0, s, nd.child_first, nd.nchild, lv, top,
                               t.nd_S.as<double4>(), t.nd_Z.as<double4>());
            TFMM_LAUNCHED();
        }
    }
    t.nd_rmax.ensure(ctx, (size_t)nn * 8);
    t.w_geo.ensure(ctx, (size_t)nn * sizeof(double4));
    t.w_top.ensure(ctx, (size_t)nn * sizeof(int4));
    t.nd_r2bits.ensure(ctx, (size_t)nn * 8);
    const double4* balls = t.balls.as<double4>();
    const bool rows = n > kWaveNodes;
    // every level holds each particle at most once
    const int64_t ub = rows ? (t.max_level + 1) * (n / kBallsFrom + n / RCH) + 1 : 0;
    t.rmax_items.ensure(ctx, (size_t)std::max<int64_t>(std::min(ub, nn + (t.max_level + 1) * (n / RCH)), 1) * 8);
    const NodePack pk{soff, ns, t.nd_rmax.as<double>(), t.w_geo.as<double4>(), t.w_top.as<int4>()};
    hipLaunchKernelGGL((rows ? rmax_kernel<16> : rmax_kernel<kWave>),
                       dim3((unsigned)cdiv(nn, TB / (rows ? 16 : kWave))), dim3(TB), 0, s, nd, nn,
                       (const double4*)t.Xm.as<double4>(), balls, (const double4*)t.nd_Z.as<double4>(), pk,
                       t.nd_r2bits.as<unsigned long long>(), t.rmax_items.as<int2>(), n_items);
    TFMM_LAUNCHED();
    if (ub > 0) {
        hipLaunchKernelGGL(rmax_items_kernel, dim3((unsigned)std::min<int64_t>(2048, cdiv(ub, TB / kWave))), dim3(TB), 0,
                           s, (const uint32_t*)n_items, (const int2*)t.rmax_items.as<int2>(), nd,
                           (const double4*)t.Xm.as<double4>(), balls, (const double4*)t.nd_Z.as<double4>(), pk,
                           t.nd_r2bits.as<unsigned long long>());
        TFMM_LAUNCHED();
        hipLaunchKernelGGL(rmax_final_kernel, dim3((unsigned)std::min<int64_t>(64, cdiv(ub, TB))), dim3(TB), 0, s,
                           (const uint32_t*)n_items, (const int2*)t.rmax_items.as<int2>(), nd,
                           (const double4*)t.nd_Z.as<double4>(), pk,
                           (const unsigned long long*)t.nd_r2bits.as<unsigned long long>());
        TFMM_LAUNCHED();
    }

    t.built = true;
}

void prepare_sources(Tree& t, int precision, hipStream_t s) {
    if (t.src_prec == precision) return;
    t.src_prec = -1;  // what is there goes when the buffer grows
    const int64_t n = t.n;
    if (precision == TFMM_MIXED32) {
        t.src4.ensure(t.ctx, (size_t)n * 16);
        hipLaunchKernelGGL(sources_kernel<float>, dim3(grid(n)), dim3(TB), 0, s, t.Xm.as<double4>(),
                           t.leaf_of.as<int32_t>(), t.nd_Z.as<double4>(), n, t.src4.as<float4>());
    } else {
        t.src4.ensure(t.ctx, (size_t)n * 32);
        hipLaunchKernelGGL(sources_kernel<double>, dim3(grid(n)), dim3(TB), 0, s, t.Xm.as<double4>(),
                           t.leaf_of.as<int32_t>(), t.nd_Z.as<double4>(), n, t.src4.as<double4>());
    }
    TFMM_LAUNCHED();
    t.src_prec = precision;
}

}  // namespace tfmm
