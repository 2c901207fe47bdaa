// Near field (P2P): exact softened pair accelerations between the particles
// of every near pair of leaves, both directions, self pairs included (the
// gradient of Eq. jia with -(r^2 + eps^2)^(-1/2)).
//
// One wavefront (= one workgroup) runs one work item: a target leaf and a piece
// of its near list (below; several wavefronts in small trees).  A chunk of nt <= 64
// target particles is laid out over the lanes as G groups of L lanes, each
// lane holding R consecutive targets (L = ceil(nt / R), G = floor(64 / L));
// group g takes every G-th staged source (the stage keeps each group's sources
// contiguous, so its loop count is uniform).  R in 1..4 is chosen per chunk to
// keep the most lanes busy (R = 1 with G replicas for small leaves, R > 1 for
// leaves of 33..64 particles), and a staged source is reused for R targets.
// Source leaves are staged into an LDS chunk already expressed in the target
// leaf's frame: the leaf-to-leaf offset Z_B - Z_A is applied in FP64 and the
// result rounded once (FP32 in the mixed path), so the inner loop is a uniform
// stream of LDS broadcasts and FMAs.  Each chunk's partial sums go into FP64
// per-lane accumulators; the groups are summed through LDS at the end.
// What bounds it (2^20 Plummer particles, 3.29e9 pairs, FP32): VALU issue.  8.8e8
// wave instructions in 1.43 ms are one per SIMD every 4 cycles; the pair formula
// alone is 13 of the 17.1 per useful pair, the rest is idle lanes of the layouts
// and staging.  The staging takes no branches (its four loads are in flight
// together), 24-bit multiplies and scalar chunk sizes, and the loops exist once
// per R: 9.27e8 instructions and 1.51 ms before that (disk of 2^22, leaves of
// 128: 2.85 -> 2.76 ms).
// A leaf's list is cut into work items of bounded source count (a leaf in a
// sparse halo can be near almost every particle); every item writes its own
// partial sums and a second kernel adds a leaf's items in order.
#include <algorithm>

#include "common.h"

namespace tfmm {
namespace {

constexpr int CH = 256;   // staged source particles per chunk
static_assert(CH + kWave <= 512, "the staging's multiplications take places below 512");
// Stage slots: G gs <= cnt + G - 1 + G <= CH + 2 kWave - 1, and a spare one.
constexpr uint32_t kSpare = CH + 2 * kWave - 1;

template <typename T>
__device__ __forceinline__ T far_away();
template <> __device__ __forceinline__ float far_away<float>() { return 1.0e18f; }
template <> __device__ __forceinline__ double far_away<double>() { return 1.0e100; }

// POT: also the potential -m_b (r^2 + eps^2)^(-1/2) into ph.
template <typename T, bool SAFE, bool POT>
__device__ __forceinline__ void interact(const typename Vec4<T>::type& s, T tx, T ty, T tz, T eps2, T& ax,
                                         T& ay, T& az, T& ph) {
    const T dx = s.x - tx, dy = s.y - ty, dz = s.z - tz;
    const T r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2)));
    T mri = T(0);
    T w = weight<POT>(r2, s.w, mri);
    if (SAFE) w = (r2 > T(0)) ? w : T(0);
    ax = fma(w, dx, ax);
    ay = fma(w, dy, ay);
    az = fma(w, dz, az);
    if constexpr (POT) ph -= (SAFE && !(r2 > T(0))) ? T(0) : mri;
}

__device__ __forceinline__ int wave_incl_scan(int v) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int u = __shfl_up(v, d, kWave);
        if (lane >= d) v += u;
    }
    return v;
}

constexpr int RMAX = 4;  // most targets per lane

// Lane layout of a target chunk: the R in 1..RMAX that keeps the most lanes
// busy (useful fraction nt * G / (64 * R)); ties go to the smaller R.
__device__ __forceinline__ void chunk_layout(int nt, int& R, int& L, int& G) {
    R = 1;
    L = nt;
    G = kWave / nt;
#pragma unroll
    for (int r = 2; r <= RMAX; ++r) {
        const int l = (nt + r - 1) / r;
        const int g = kWave / l;
        if (g * R > G * r) {  // nt g / r > nt G / R
            R = r;
            L = l;
            G = g;
        }
    }
}

// Interactions of one staged chunk for a lane's R targets: the ng sources its
// group owns, stored contiguously from src (the loop count is the same for
// every lane, so the loop runs on scalar registers).
template <typename T, bool SAFE, bool POT, int R>
__device__ __forceinline__ void consume(const typename Vec4<T>::type* src, int ng, const T* tx, const T* ty,
                                        const T* tz, T eps2, T* sx, T* sy, T* sz, T* sp) {
    constexpr int U = (R >= 4) ? 1 : 4 / R;
    const int nmain = ng / U * U;
    int i = 0;
    for (; i < nmain; i += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const typename Vec4<T>::type v = src[i + u];
#pragma unroll
            for (int r = 0; r < R; ++r)
                interact<T, SAFE, POT>(v, tx[r], ty[r], tz[r], eps2, sx[r], sy[r], sz[r], sp[r]);
        }
    }
    for (; i < ng; ++i) {
        const typename Vec4<T>::type v = src[i];
#pragma unroll
        for (int r = 0; r < R; ++r) interact<T, SAFE, POT>(v, tx[r], ty[r], tz[r], eps2, sx[r], sy[r], sz[r], sp[r]);
    }
}

// Staging constants of a chunk of G groups with ng sources each: source c has
// stage slot (c % G) gs + c / G = c gs - (c / G) (G gs - 1).  c / G for c < CH +
// kWave is (c gm) >> 16, gm = ceil(2^16 / G): exact while c (gm G - 2^16) < 2^16,
// i.e. for every c below 1040.  The masks tell the compiler that 24-bit
// multiplies do: a 32-bit one takes four times the issue slots.
struct Slots {
    uint32_t gs, gm, k;
    __device__ __forceinline__ Slots(int G, int ng)
        : gs((uint32_t)(ng | 1) & 0x1ff), gm((uint32_t)((65536 + G - 1) / G) & 0x1ffff),
          k(((uint32_t)G * gs - 1u) & 0x7fff) {}
    __device__ __forceinline__ uint32_t operator()(uint32_t c) const {
        const uint32_t q = ((c & 0x1ff) * gm) >> 16;
        return (c & 0x1ff) * gs - q * k;
    }
};

// One source leaf of the window: the offset of its centre from the target
// leaf's, and its first particle less its place in the window (so that source
// s of the window is particle s + delta).
struct Entry {
    double x, y, z;
    int delta, pad;
};

// Fills lane's entry of the window of ne list entries from list position qb;
// start[lane] is its first source in the window (the lanes past ne get a place
// past every source).  Returns the window's sources.
__device__ __forceinline__ int load_window(const int32_t* __restrict__ src, const int32_t* __restrict__ first,
                                           const int32_t* __restrict__ count, const double4* __restrict__ Z,
                                           uint32_t qb, int ne, int lane, const double4& za, int* start,
                                           Entry* entry) {
    int nb = 0, f = 0;
    Entry e{0.0, 0.0, 0.0, 0, 0};
    if (lane < ne) {
        const int32_t B = src[qb + lane];
        const double4 zb = Z[B];
        nb = count[B];
        f = first[B];
        e.x = zb.x - za.x;
        e.y = zb.y - za.y;
        e.z = zb.z - za.z;
    }
    const int incl = wave_incl_scan(nb);
    e.delta = f - (incl - nb);
    entry[lane] = e;
    start[lane] = (lane < ne) ? incl - nb : 0x7fffffff;
    if (lane == 0) start[kWave] = 0x7fffffff;
    return __builtin_amdgcn_readlane(incl, kWave - 1);  // scalar: so are the chunk sizes
}

// Stages sources c0 .. c0 + cnt - 1 of the window whose entries are in the
// tables, padded to a multiple of G; group g owns sources g, g + G, ...,
// stored contiguously at g * gs (gs = ng | 1 is odd, so the groups' reads of
// one step fall in distinct LDS banks).  Returns ng, the sources per group.
template <typename T>
__device__ __forceinline__ int stage_chunk(const typename Vec4<T>::type* __restrict__ P, int lane, int c0, int cnt,
                                           int G, const int* start, const Entry* entry,
                                           typename Vec4<T>::type* stage) {
    using V4 = typename Vec4<T>::type;
    constexpr int SPL = CH / kWave;  // staged sources per lane per chunk
    // the lane takes the consecutive sources c0 + SPL lane + k (past the last
    // one, that one again); the entry of the first by binary search, then at
    // most one step per source (every entry holds at least one source).  No
    // branches: the four loads are in flight together.
    int ent[SPL];
    V4 v[SPL];
    {
        const int last = c0 + cnt - 1;
        int sidx = c0 + SPL * lane;
        sidx = sidx < last ? sidx : last;
        int lo = 0;
#pragma unroll
        for (int st = kWave / 2; st > 0; st >>= 1) lo += start[lo + st] <= sidx ? st : 0;
#pragma unroll
        for (int k = 0; k < SPL; ++k) {
            if (k > 0) {
                sidx = sidx < last ? sidx + 1 : last;
                lo += start[lo + 1] <= sidx ? 1 : 0;
            }
            ent[k] = lo;
            v[k] = P[sidx + entry[lo].delta];
        }
    }
    const int cp = (cnt + G - 1) / G * G;
    const int ng = cp / G;
    const Slots slot(G, ng);
#pragma unroll
    for (int k = 0; k < SPL; ++k) {
        const int c = SPL * lane + k;
        const Entry& e = entry[ent[k]];
        V4 w;
        w.x = (T)((double)v[k].x + e.x);
        w.y = (T)((double)v[k].y + e.y);
        w.z = (T)((double)v[k].z + e.z);
        w.w = v[k].w;
        stage[c < cnt ? slot((uint32_t)c) : kSpare] = w;
    }
    // pads (their slots are distinct from the sources')
    if (cnt + lane < cp) {
        V4 pad;
        pad.x = far_away<T>();
        pad.y = far_away<T>();
        pad.z = far_away<T>();
        pad.w = T(0);
        stage[slot((uint32_t)(cnt + lane))] = pad;
    }
    return ng;
}

// One target chunk (targets tc .. tc + nt - 1 of the leaf, laid out as G
// groups of L lanes with R targets each) against the sources of list entries
// q0 .. q1 - 1.  The sums of a staged chunk are added to FP64 accumulators.
template <typename T, bool SAFE, bool POT, int R>
__device__ __forceinline__ void target_chunk(int nt, int L, int G, uint32_t q0, uint32_t q1, const double4& za,
                                             const int32_t* __restrict__ first, const int32_t* __restrict__ count,
                                             const int32_t* __restrict__ src, const double4* __restrict__ Z,
                                             const typename Vec4<T>::type* __restrict__ P,
                                             const typename Vec4<T>::type* __restrict__ tgt, T eps2,
                                             typename Vec4<T>::type* stage, int* start, Entry* entry,
                                             double (*red)[kWave], double* __restrict__ out,
                                             double* __restrict__ pout) {
    using V4 = typename Vec4<T>::type;
    const int lane = threadIdx.x;
    const int l = lane % L;
    const int g = lane / L;
    const bool act = g < G;
    // the lane's targets l R + r; slots past nt repeat a valid target and are dropped
    T tx[R], ty[R], tz[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int ti = l * R + r;
        ti = ti < nt ? ti : nt - 1;
        const V4 me = tgt[ti];
        tx[r] = me.x;
        ty[r] = me.y;
        tz[r] = me.z;
    }
    double ax[R], ay[R], az[R], ap[R];
#pragma unroll
    for (int r = 0; r < R; ++r) ax[r] = ay[r] = az[r] = ap[r] = 0.0;

    for (uint32_t qb = q0; qb < q1; qb += kWave) {
        const int ne = (int)((q1 - qb) < (uint32_t)kWave ? (q1 - qb) : (uint32_t)kWave);
        const int total = load_window(src, first, count, Z, qb, ne, lane, za, start, entry);
        __syncthreads();
        for (int c0 = 0; c0 < total; c0 += CH) {
            const int cnt = (total - c0) < CH ? (total - c0) : CH;
            const int ng = stage_chunk<T>(P, lane, c0, cnt, G, start, entry, stage);
            __syncthreads();
            T sx[R], sy[R], sz[R], sp[R];
#pragma unroll
            for (int r = 0; r < R; ++r) sx[r] = sy[r] = sz[r] = sp[r] = T(0);
            if (act) consume<T, SAFE, POT, R>(stage + g * (ng | 1), ng, tx, ty, tz, eps2, sx, sy, sz, sp);
#pragma unroll
            for (int r = 0; r < R; ++r) {  // inactive lanes add zeros
                ax[r] += (double)sx[r];
                ay[r] += (double)sy[r];
                az[r] += (double)sz[r];
                if constexpr (POT) ap[r] += (double)sp[r];
            }
            __syncthreads();
        }
    }

    // target t = l R + r sits in slot r of lanes l, l + L, ..., one per group;
    // slot by slot, through LDS
    const int tl = lane / R, tr = lane % R;
    double fx = 0.0, fy = 0.0, fz = 0.0, fp = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        red[0][lane] = ax[r];
        red[1][lane] = ay[r];
        red[2][lane] = az[r];
        if constexpr (POT) red[POT ? 3 : 0][lane] = ap[r];
        __syncthreads();
        if (lane < nt && tr == r) {
            for (int q = 0; q < G; ++q) {
                fx += red[0][q * L + tl];
                fy += red[1][q * L + tl];
                fz += red[2][q * L + tl];
                if constexpr (POT) fp += red[POT ? 3 : 0][q * L + tl];
            }
        }
        __syncthreads();
    }
    if (lane < nt) {
        out[3 * lane] = fx;
        out[3 * lane + 1] = fy;
        out[3 * lane + 2] = fz;
        if constexpr (POT) pout[lane] = fp;
    }
}

// POT: the near-field potential too (-sum m_b (r^2 + eps^2)^(-1/2), the
// particle's own term included when eps > 0; the caller removes it).
template <typename T, bool SAFE, bool POT>
__global__ __launch_bounds__(kWave) void p2p_kernel(const int32_t* __restrict__ it_leaf,
                                                    const uint32_t* __restrict__ it_q0,
                                                    const uint32_t* __restrict__ it_q1,
                                                    const uint32_t* __restrict__ it_pbase,
                                                    const int32_t* __restrict__ first,
                                                    const int32_t* __restrict__ count,
                                                    const int32_t* __restrict__ src,
                                                    const double4* __restrict__ Z,
                                                    const typename Vec4<T>::type* __restrict__ P, T eps2,
                                                    const int32_t* __restrict__ leaf_nitems,
                                                    double* __restrict__ partial, double* __restrict__ near,
                                                    double* __restrict__ partial_pot,
                                                    double* __restrict__ near_pot) {
    using V4 = typename Vec4<T>::type;
    __shared__ V4 stage[CH + 2 * kWave];
    __shared__ int start[kWave + 1];
    __shared__ Entry entry[kWave];
    __shared__ double red[POT ? 4 : 3][kWave];
    // work items (in target leaf order) in chunks of 32 per XCD
    const uint32_t blk = xcd_block<32>(blockIdx.x, gridDim.x);
    const int32_t A = it_leaf[blk];
    const int32_t fa = first[A], na = count[A];
    const double4 za = Z[A];
    const uint32_t q0 = it_q0[blk], q1 = it_q1[blk];
    // a leaf served by one item writes the result, otherwise its own partial slot
    const bool whole = leaf_nitems[A] == 1;
    double* out = whole ? near + 3 * (int64_t)fa : partial + 3 * (int64_t)it_pbase[blk];
    double* pout = nullptr;
    if constexpr (POT) pout = whole ? near_pot + fa : partial_pot + it_pbase[blk];

    for (int32_t tc = 0; tc < na; tc += kWave) {
        const int nt = (na - tc) < kWave ? (na - tc) : kWave;
        int R, L, G;
        chunk_layout(nt, R, L, G);
        const V4* tgt = P + fa + tc;
        // one copy of the loops per R: with the choice inside them the compiler
        // copied all accumulators at every chunk
        switch (R) {
            case 1:
                target_chunk<T, SAFE, POT, 1>(nt, L, G, q0, q1, za, first, count, src, Z, P, tgt, eps2, stage, start,
                                              entry, red, out + 3 * tc, pout + tc);
                break;
            case 2:
                target_chunk<T, SAFE, POT, 2>(nt, L, G, q0, q1, za, first, count, src, Z, P, tgt, eps2, stage, start,
                                              entry, red, out + 3 * tc, pout + tc);
                break;
            case 3:
                target_chunk<T, SAFE, POT, 3>(nt, L, G, q0, q1, za, first, count, src, Z, P, tgt, eps2, stage, start,
                                              entry, red, out + 3 * tc, pout + tc);
                break;
            default:
                target_chunk<T, SAFE, POT, 4>(nt, L, G, q0, q1, za, first, count, src, Z, P, tgt, eps2, stage, start,
                                              entry, red, out + 3 * tc, pout + tc);
                break;
        }
    }
}

// The same work item run by a workgroup of W wavefronts, for trees with too few
// items to fill the device with one wavefront each.  Wavefront w takes chunks
// w, w + W, ... of every entry window; a round's FP32 (FP64) chunk sums go
// through LDS and are added to the FP64 accumulators in chunk order, so the
// result is the single-wavefront kernel's bit for bit.  A lane's 3 R sums
// (4 R with the potential) are accumulated by the W wavefronts together, slot k
// by wavefront k % W.
template <typename T, bool SAFE, bool POT, int W>
__global__ __launch_bounds__(W* kWave) void p2p_block_kernel(const int32_t* __restrict__ it_leaf,
                                                             const uint32_t* __restrict__ it_q0,
                                                             const uint32_t* __restrict__ it_q1,
                                                             const uint32_t* __restrict__ it_pbase,
                                                             const int32_t* __restrict__ first,
                                                             const int32_t* __restrict__ count,
                                                             const int32_t* __restrict__ src,
                                                             const double4* __restrict__ Z,
                                                             const typename Vec4<T>::type* __restrict__ P, T eps2,
                                                             const int32_t* __restrict__ leaf_nitems,
                                                             double* __restrict__ partial, double* __restrict__ near,
                                                             double* __restrict__ partial_pot,
                                                             double* __restrict__ near_pot) {
    using V4 = typename Vec4<T>::type;
    constexpr int ND = POT ? 4 : 3;                 // components per target
    constexpr int NS = ND * RMAX;                   // sums per lane
    constexpr int NA = (NS + W - 1) / W;            // of which a wavefront accumulates
    constexpr int SW = (CH + 2 * kWave) * (int)(sizeof(V4) / sizeof(T));  // a wavefront's stage, in scalars
    static_assert(NS * kWave <= SW && NS * kWave * 8 <= W * SW * (int)sizeof(T), "sums fit the stage");
    // staged sources; the chunk sums and the final sums reuse the space
    __shared__ __attribute__((aligned(32))) T stage_all[W][SW];
    __shared__ int start[kWave + 1];
    __shared__ Entry entry[kWave];
    __shared__ int s_total;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    V4* stage = reinterpret_cast<V4*>(stage_all[wv]);
    T* csum = stage_all[wv];
    double* red = reinterpret_cast<double*>(&stage_all[0][0]);
    const uint32_t blk = xcd_block<32>(blockIdx.x, gridDim.x);
    const int32_t A = it_leaf[blk];
    const int32_t fa = first[A], na = count[A];
    const double4 za = Z[A];
    const uint32_t q0 = it_q0[blk], q1 = it_q1[blk];
    const bool whole = leaf_nitems[A] == 1;
    double* out = whole ? near + 3 * (int64_t)fa : partial + 3 * (int64_t)it_pbase[blk];
    double* pout = nullptr;
    if constexpr (POT) pout = whole ? near_pot + fa : partial_pot + it_pbase[blk];

    for (int32_t tc = 0; tc < na; tc += kWave) {
        const int nt = (na - tc) < kWave ? (na - tc) : kWave;
        int R, L, G;
        chunk_layout(nt, R, L, G);
        const int l = lane % L;
        const int g = lane / L;
        const bool act = g < G;
        T tx[RMAX], ty[RMAX], tz[RMAX];
#pragma unroll
        for (int r = 0; r < RMAX; ++r) {
            int ti = l * R + r;
            ti = ti < nt ? ti : nt - 1;
            const V4 me = P[fa + tc + ti];
            tx[r] = me.x;
            ty[r] = me.y;
            tz[r] = me.z;
        }
        double acc[NA];
#pragma unroll
        for (int k = 0; k < NA; ++k) acc[k] = 0.0;

        for (uint32_t qb = q0; qb < q1; qb += kWave) {
            const int ne = (int)((q1 - qb) < (uint32_t)kWave ? (q1 - qb) : (uint32_t)kWave);
            if (wv == 0) {
                const int tot = load_window(src, first, count, Z, qb, ne, lane, za, start, entry);
                if (lane == 0) s_total = tot;
            }
            __syncthreads();
            const int total = __builtin_amdgcn_readfirstlane(s_total);

            for (int cb = 0; cb < total; cb += W * CH) {
                const int c0 = cb + wv * CH;
                int ng = 0;
                if (c0 < total) {
                    const int cnt = (total - c0) < CH ? (total - c0) : CH;
                    ng = stage_chunk<T>(P, lane, c0, cnt, G, start, entry, stage);
                }
                __syncthreads();
                if (c0 < total) {
                    const V4* sp0 = stage + g * (ng | 1);
                    T sx[RMAX], sy[RMAX], sz[RMAX], sp[RMAX];
#pragma unroll
                    for (int r = 0; r < RMAX; ++r) sx[r] = sy[r] = sz[r] = sp[r] = T(0);
                    if (act) {
                        switch (R) {
                            case 1: consume<T, SAFE, POT, 1>(sp0, ng, tx, ty, tz, eps2, sx, sy, sz, sp); break;
                            case 2: consume<T, SAFE, POT, 2>(sp0, ng, tx, ty, tz, eps2, sx, sy, sz, sp); break;
                            case 3: consume<T, SAFE, POT, 3>(sp0, ng, tx, ty, tz, eps2, sx, sy, sz, sp); break;
                            default: consume<T, SAFE, POT, 4>(sp0, ng, tx, ty, tz, eps2, sx, sy, sz, sp); break;
                        }
                    }
#pragma unroll
                    for (int r = 0; r < RMAX; ++r) {
                        if (r < R) {
                            csum[(ND * r) * kWave + lane] = sx[r];
                            csum[(ND * r + 1) * kWave + lane] = sy[r];
                            csum[(ND * r + 2) * kWave + lane] = sz[r];
                            if constexpr (POT) csum[(ND * r + 3) * kWave + lane] = sp[r];
                        }
                    }
                }
                __syncthreads();
                // the round's chunks in order
                const int nc = (total - cb + CH - 1) / CH < W ? (total - cb + CH - 1) / CH : W;
#pragma unroll
                for (int k = 0; k < NA; ++k) {
                    const int slot = wv + k * W;
                    if (slot < ND * R)
                        for (int c = 0; c < nc; ++c) acc[k] += (double)stage_all[c][slot * kWave + lane];
                }
                __syncthreads();  // the next round stages, the next window rewrites the tables
            }
        }

#pragma unroll
        for (int k = 0; k < NA; ++k) {
            const int slot = wv + k * W;
            if (slot < ND * R) red[slot * kWave + lane] = acc[k];
        }
        __syncthreads();
        // component d of target t = l R + r: slot ND r + d of lanes l, l + L, ...
        const int tl = lane / R, tr = lane % R;
        for (int d = wv; d < ND; d += W) {
            if (lane < nt) {
                double f = 0.0;
                for (int q = 0; q < G; ++q) f += red[(ND * tr + d) * kWave + q * L + tl];
                const int64_t j = (int64_t)(tc + lane);
                if (POT && d == 3) pout[j] = f;
                else out[3 * j + d] = f;
            }
        }
        __syncthreads();
    }
}

// Leaves served by several items (listed in multi_leaf, in any order): one
// wavefront per such leaf adds the items' partial sums in item order.  The
// grid is an upper bound of the list length; the surplus wavefronts exit.
template <bool POT>
__global__ __launch_bounds__(kWave) void p2p_reduce_kernel(const int32_t* __restrict__ multi_leaf,
                                                           const uint32_t* __restrict__ multi_count,
                                                           const int32_t* __restrict__ leaf_item0,
                                                           const int32_t* __restrict__ leaf_nitems,
                                                           const int32_t* __restrict__ first,
                                                           const int32_t* __restrict__ count,
                                                           const uint32_t* __restrict__ it_pbase,
                                                           const double* __restrict__ partial,
                                                           double* __restrict__ near,
                                                           const double* __restrict__ partial_pot,
                                                           double* __restrict__ near_pot) {
    if (blockIdx.x >= *multi_count) return;
    const int32_t L = multi_leaf[blockIdx.x];
    const int32_t ni = leaf_nitems[L], i0 = leaf_item0[L];
    const int32_t fa = first[L], na = count[L];
    constexpr int B = 8;  // items whose rows are loaded together (sums stay in item order)
    for (int32_t r = threadIdx.x; r < na; r += kWave) {
        double sx = 0.0, sy = 0.0, sz = 0.0, sp = 0.0;
        for (int32_t i = 0; i < ni; i += B) {
            int64_t row[B];
#pragma unroll
            for (int u = 0; u < B; ++u) row[u] = i + u < ni ? (int64_t)it_pbase[i0 + i + u] + r : 0;
            double v[B][4];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                if (i + u < ni) {
                    const double* p = partial + 3 * row[u];
                    v[u][0] = p[0];
                    v[u][1] = p[1];
                    v[u][2] = p[2];
                    if constexpr (POT) v[u][3] = partial_pot[row[u]];
                }
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                if (i + u < ni) {
                    sx += v[u][0];
                    sy += v[u][1];
                    sz += v[u][2];
                    if constexpr (POT) sp += v[u][3];
                }
            }
        }
        near[3 * (int64_t)(fa + r)] = sx;
        near[3 * (int64_t)(fa + r) + 1] = sy;
        near[3 * (int64_t)(fa + r) + 2] = sz;
        if constexpr (POT) near_pot[fa + r] = sp;
    }
}

// Trees of at most block_items() items run each item by a workgroup of four
// wavefronts, of at most kBlockItems8 by eight: one wavefront per item leaves
// many of the 1024 SIMDs idle or with a single wavefront there, and the pass
// lasts as long as its longest items.  Steps on one MI355X, one / four / eight
// wavefronts per item: ball of 2048 (67 items) 409 / 362 / 365 us, Plummer
// 5000 (300 items, four steps) 2660 / 2385 / 2314, Plummer 20011 in FP64 (2.9e3
// items) 783 / 711 / 812, 16 sets of 131072 particles (5.7e3 items) 890 / 786 /
// 832; one / four: Plummer 10^5 (conserving, order 4) 920 / 850, 2^18 (1.7e4 items)
// 1256 / 1228.  Past that the rounds' barriers cost more than the shorter tail
// gives: balls of 2e5 and 3e5 (1.7e4 and 1.8e4 items) even, Plummer 3.3e5 1379 /
// 1440, 4.8e5 1786 / 1880; in FP64, with 12 wavefronts per compute unit, already
// 1.3e5 even and 2^18 2097 / 2178.
template <typename T>
constexpr int64_t block_items() { return sizeof(T) == 4 ? 18432 : 8192; }  // 72, 32 per compute unit
constexpr int64_t kBlockItems8 = 512;

template <typename T, bool POT>
void launch(Tree& t, double eps2, hipStream_t s) {
    using V4 = typename Vec4<T>::type;
    const int64_t ni = t.n_items;
    if (ni <= 0) return;
    auto run = [&](auto kern, int waves) {
        hipLaunchKernelGGL(kern, dim3((unsigned)ni), dim3(waves * kWave), 0, s, t.it_leaf.as<int32_t>(),
                           t.it_q0.as<uint32_t>(), t.it_q1.as<uint32_t>(), t.it_pbase.as<uint32_t>(),
                           t.nd_first.as<int32_t>(), t.nd_count.as<int32_t>(), t.p2p_src.as<int32_t>(),
                           t.nd_Z.as<double4>(), t.src4.as<V4>(), (T)eps2, t.leaf_nitems.as<int32_t>(),
                           t.partial.as<double>(), t.near3.as<double>(),
                           POT ? t.partial_pot.as<double>() : nullptr, POT ? t.near_pot.as<double>() : nullptr);
        TFMM_LAUNCHED();
    };
    const bool safe = !(eps2 > 0.0);
    if (ni <= kBlockItems8) {
        if (safe) run(p2p_block_kernel<T, true, POT, 8>, 8);
        else run(p2p_block_kernel<T, false, POT, 8>, 8);
    } else if (ni <= block_items<T>()) {
        if (safe) run(p2p_block_kernel<T, true, POT, 4>, 4);
        else run(p2p_block_kernel<T, false, POT, 4>, 4);
    } else {
        if (safe) run(p2p_kernel<T, true, POT>, 1);
        else run(p2p_kernel<T, false, POT>, 1);
    }
}

template <bool POT>
void launch_reduce(Tree& t, hipStream_t s) {
    const int64_t ni = t.n_items;
    if (ni <= 0) return;
    double* ppot = POT ? t.partial_pot.as<double>() : nullptr;
    double* npot = POT ? t.near_pot.as<double>() : nullptr;
    // every leaf has at least one item, so at most n_items - n_leaves leaves have several
    const int64_t nmulti = ni - t.n_leaves;
    if (nmulti > 0) {
        hipLaunchKernelGGL((p2p_reduce_kernel<POT>), dim3((unsigned)nmulti), dim3(kWave), 0, s,
                           t.multi_leaf.as<int32_t>(), t.multi_count, t.leaf_item0.as<int32_t>(),
                           t.leaf_nitems.as<int32_t>(), t.nd_first.as<int32_t>(), t.nd_count.as<int32_t>(),
                           t.it_pbase.as<uint32_t>(), t.partial.as<double>(), t.near3.as<double>(),
                           (const double*)ppot, npot);
        TFMM_LAUNCHED();
    }
}

}  // namespace

// The partial sums of leaves whose near list was cut into several items
// (after run_p2p on the same stream).
void run_p2p_reduce(Tree& t, bool with_pot, hipStream_t s) {
    if (with_pot) launch_reduce<true>(t, s);
    else launch_reduce<false>(t, s);
}

void run_p2p(Tree& t, int precision, double eps2, bool with_pot, hipStream_t s) {
    t.near3.ensure(t.ctx, (size_t)t.n * 24);
    t.partial.ensure(t.ctx, (size_t)std::max<int64_t>(t.n_partial, 1) * 24);
    if (with_pot) {
        t.near_pot.ensure(t.ctx, (size_t)t.n * 8);
        t.partial_pot.ensure(t.ctx, (size_t)std::max<int64_t>(t.n_partial, 1) * 8);
        if (precision == TFMM_MIXED32) launch<float, true>(t, eps2, s);
        else launch<double, true>(t, eps2, s);
    } else {
        if (precision == TFMM_MIXED32) launch<float, false>(t, eps2, s);
        else launch<double, false>(t, eps2, s);
    }
}

}  // namespace tfmm
