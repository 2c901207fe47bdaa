// Multipole moments of every node in FP64 (the paper's step (i), Sec. 2).
//
// Raw Cartesian moments about the node's centre of mass, M_k = sum_b m_b y_b^k
// with y_b = Y_b - Z_B and |k| <= p (the monopole, quadrupole, octopole, ...
// of Eqs. quad_mom, octo_mom, hexa_mom before their traces are removed; with
// a softened kernel the traces matter), are stored in the form the M2L
// kernels contract with:
//     W_k = (-1)^|k| M_k / k! = sum_b m_b (-y_b)^k / k!.
// Leaves sum over their particles (P2M).  Inner nodes shift their children
// exactly (M2M): with y' = y + d_c, d_c = Z_c - Z_P,
//     W_k(P) = sum_c sum_{i + j = k} W_i(c) (-d_c)^j / j!.
// FP64 throughout; an FP32 copy feeds the mixed-precision M2L.
#include "common.h"
#include "expansions_gen.h"

namespace tfmm {
namespace {

constexpr int TB = 256;
constexpr int LPL = 4;  // lanes per leaf
constexpr int LPN = 8;  // lanes per inner node: one per child

// Writes a node's moments, summed over its group of LANES lanes (x: this
// lane's place), quads of coefficients dealt to the lanes.
template <int P, int LANES>
__device__ __forceinline__ void write_moments(const double* w, int32_t node, int x, double* __restrict__ W64,
                                              float* __restrict__ W32) {
    constexpr int NC = Expansion<P>::NC;
    constexpr int NCP = (NC + 3) / 4 * 4;
    double4* o64 = reinterpret_cast<double4*>(W64 + (int64_t)node * NCP);
    float4* o32 = reinterpret_cast<float4*>(W32 + (int64_t)node * NCP);
#pragma unroll
    for (int q = 0; q < NCP / 4; ++q) {
        double4 v;
        v.x = group_sum<LANES>(w[4 * q]);
        v.y = 4 * q + 1 < NC ? group_sum<LANES>(w[4 * q + 1]) : 0.0;
        v.z = 4 * q + 2 < NC ? group_sum<LANES>(w[4 * q + 2]) : 0.0;
        v.w = 4 * q + 3 < NC ? group_sum<LANES>(w[4 * q + 3]) : 0.0;
        if (x == q % LANES) {
            o64[q] = v;
            o32[q] = make_float4((float)v.x, (float)v.y, (float)v.z, (float)v.w);
        }
    }
}

template <int P>
__global__ __launch_bounds__(TB) void p2m_kernel(int64_t n_leaves, const int32_t* __restrict__ leaves,
                                                 const int32_t* __restrict__ first,
                                                 const int32_t* __restrict__ count,
                                                 const double4* __restrict__ Xm, const double4* __restrict__ Z,
                                                 double* __restrict__ W64, float* __restrict__ W32) {
    using E = Expansion<P>;
    constexpr int NC = E::NC;
    const int64_t i = ((int64_t)blockIdx.x * TB + threadIdx.x) / LPL;
    const int x = threadIdx.x % LPL;
    const bool live = i < n_leaves;  // the lanes of a group agree; every lane takes part in the sums
    const int32_t node = leaves[live ? i : 0];
    const double4 z = Z[node];
    double w[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) w[k] = 0.0;
    const int32_t s0 = first[node], s1 = live ? s0 + count[node] : s0;
    for (int32_t s = s0 + x; s < s1; s += 2 * LPL) {
        const bool two = s + LPL < s1;
        const double4 p = Xm[s], q = Xm[two ? s + LPL : s];
        E::p2m(p.w, z.x - p.x, z.y - p.y, z.z - p.z, w);
        if (two) E::p2m(q.w, z.x - q.x, z.y - q.y, z.z - q.z, w);
    }
    if (live) write_moments<P, LPL>(w, node, x, W64, W32);
}

// One inner node: lane x shifts child x, the group adds up.
template <int P>
__device__ __forceinline__ void m2m_node(int32_t node, int x, bool live, const int32_t* __restrict__ child_first,
                                         const int32_t* __restrict__ nchild, const double4* __restrict__ Z,
                                         double* __restrict__ W64, float* __restrict__ W32) {
    using E = Expansion<P>;
    constexpr int NC = E::NC;
    constexpr int NCP = (NC + 3) / 4 * 4;
    const int32_t nc = live ? nchild[node] : 0;
    double w[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) w[k] = 0.0;
    if (x < nc) {
        const int32_t c = child_first[node] + x;
        const double4 z = Z[node], zc = Z[c];
        E::m2m(W64 + (int64_t)c * NCP, z.x - zc.x, z.y - zc.y, z.z - zc.z, w);
    }
    if (nc > 0) write_moments<P, LPN>(w, node, x, W64, W32);  // leaves: P2M
}

template <int P>
__global__ __launch_bounds__(TB) void m2m_kernel(int32_t lb, int32_t le, const int32_t* __restrict__ child_first,
                                                 const int32_t* __restrict__ nchild,
                                                 const double4* __restrict__ Z, double* __restrict__ W64,
                                                 float* __restrict__ W32) {
    const int32_t node = lb + (int32_t)((blockIdx.x * TB + threadIdx.x) / LPN);
    m2m_node<P>(node < le ? node : lb, threadIdx.x % LPN, node < le, child_first, nchild, Z, W64, W32);
}

// Consecutive levels top..bottom of at most kFewNodes nodes each, in one block.
constexpr int kFewNodes = 2 * TB / LPN;
struct LevelBounds {
    int32_t b[kLevels + 2];
};
template <int P>
__global__ __launch_bounds__(TB) void m2m_levels_kernel(LevelBounds lv, int bottom, int top,
                                                        const int32_t* __restrict__ child_first,
                                                        const int32_t* __restrict__ nchild,
                                                        const double4* __restrict__ Z, double* W64, float* W32) {
    for (int L = bottom; L >= top; --L) {
        const int32_t lb = lv.b[L], le = lv.b[L + 1];
        for (int32_t base = lb; base < le; base += TB / LPN) {
            const int32_t node = base + (int32_t)(threadIdx.x / LPN);
            m2m_node<P>(node < le ? node : lb, threadIdx.x % LPN, node < le, child_first, nchild, Z, W64, W32);
        }
        __syncthreads();
    }
}

template <int P>
void run(Tree& t, hipStream_t s) {
    hipLaunchKernelGGL(p2m_kernel<P>, dim3((unsigned)cdiv(t.n_leaves * LPL, TB)), dim3(TB), 0, s, t.n_leaves,
                       t.leaves.as<int32_t>(), t.nd_first.as<int32_t>(), t.nd_count.as<int32_t>(),
                       t.Xm.as<double4>(), t.nd_Z.as<double4>(), t.W64.as<double>(), t.W32.as<float>());
    TFMM_LAUNCHED();
    LevelBounds lv{};
    for (int L = 0; L <= t.max_level + 1; ++L) lv.b[L] = (int32_t)t.level_begin[L];
    auto nodes = [&](int L) { return lv.b[L + 1] - lv.b[L]; };
    for (int L = t.max_level - 1; L >= 0; --L) {
        int top = L;
        while (top > 0 && nodes(L) <= kFewNodes && nodes(top - 1) <= kFewNodes) --top;
        if (top < L) {
            hipLaunchKernelGGL(m2m_levels_kernel<P>, dim3(1), dim3(TB), 0, s, lv, L, top,
                               t.nd_child_first.as<int32_t>(), t.nd_nchild.as<int32_t>(), t.nd_Z.as<double4>(),
                               t.W64.as<double>(), t.W32.as<float>());
            L = top;
        } else {
            hipLaunchKernelGGL(m2m_kernel<P>, dim3((unsigned)cdiv((int64_t)nodes(L) * LPN, TB)), dim3(TB), 0, s,
                               lv.b[L], lv.b[L + 1], t.nd_child_first.as<int32_t>(), t.nd_nchild.as<int32_t>(),
                               t.nd_Z.as<double4>(), t.W64.as<double>(), t.W32.as<float>());
        }
        TFMM_LAUNCHED();
    }
}

}  // namespace

void moments_room(Tree& t, int p) {
    if (t.mom_p == p) return;
    t.mom_p = -1;  // what is there goes when the buffers grow
    const int NCP = (int)round_up(c_le(p), 4);
    const int64_t nn = t.n_nodes;
    t.W64.ensure(t.ctx, (size_t)nn * NCP * 8);
    t.W32.ensure(t.ctx, (size_t)nn * NCP * 4);
}

// After moments_room.
void compute_moments(Tree& t, int p, hipStream_t s) {
    if (t.mom_p == p) return;
    switch (p) {
        case 1: run<1>(t, s); break;
        case 2: run<2>(t, s); break;
        case 3: run<3>(t, s); break;
        case 4: run<4>(t, s); break;
        case 5: run<5>(t, s); break;
        case 6: run<6>(t, s); break;
        case 7: run<7>(t, s); break;
        case 8: run<8>(t, s); break;
        default: fail(TFMM_EINVAL, "p must be in 1..8");
    }
    t.mom_p = p;
}

}  // namespace tfmm
