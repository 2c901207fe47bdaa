// Kick-drift-kick leapfrog on state resident in device memory (FP64).
//
// The paper evolves a self-gravitating star with FMM gravity (Sec. 4) and
// reads off the angular momentum over time; here the gravity-only analogue:
//   v += (F / m) dt/2;  x += v dt;  F = F(x);  v += (F / m) dt/2.
// Both the kick and the drift are exact elementwise updates in FP64; the
// tree is rebuilt from the drifted positions before every force evaluation.
#include "common.h"

namespace tfmm {
namespace {

constexpr int KB = 256;

__device__ __forceinline__ void kick(double* v, const double* __restrict__ force, int64_t i, double s) {
#pragma unroll
    for (int d = 0; d < 3; ++d) v[d] = fma(force[3 * i + d], s, v[d]);
}

__global__ __launch_bounds__(KB) void kick_kernel(int64_t n, double* __restrict__ vel,
                                                  const double* __restrict__ force,
                                                  const double* __restrict__ mass, double h) {
    const int64_t i = (int64_t)blockIdx.x * KB + threadIdx.x;
    if (i >= n) return;
    double v[3] = {vel[3 * i], vel[3 * i + 1], vel[3 * i + 2]};
    kick(v, force, i, h / mass[i]);
#pragma unroll
    for (int d = 0; d < 3; ++d) vel[3 * i + d] = v[d];
}

// The kick that ends a step (if both), the one that starts the next, and its
// drift: one launch between two force evaluations instead of three (four steps
// of 5000 particles, with the smaller sort and the single r_max launch of such sets,
// 1690 -> 1657 us).
__global__ __launch_bounds__(KB) void kick_drift_kernel(int64_t n, double* __restrict__ pos,
                                                        double* __restrict__ vel,
                                                        const double* __restrict__ force,
                                                        const double* __restrict__ mass, double h, double dt,
                                                        int both) {
    const int64_t i = (int64_t)blockIdx.x * KB + threadIdx.x;
    if (i >= n) return;
    const double s = h / mass[i];
    double v[3] = {vel[3 * i], vel[3 * i + 1], vel[3 * i + 2]};
    if (both) kick(v, force, i, s);
    kick(v, force, i, s);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        vel[3 * i + d] = v[d];
        pos[3 * i + d] = fma(v[d], dt, pos[3 * i + d]);
    }
}

}  // namespace

void run_kick(int64_t n, double* vel, const double* force, const double* mass, double h, hipStream_t s) {
    hipLaunchKernelGGL(kick_kernel, dim3((unsigned)cdiv(n, KB)), dim3(KB), 0, s, n, vel, force, mass, h);
    TFMM_LAUNCHED();
}

void run_kick_drift(int64_t n, double* pos, double* vel, const double* force, const double* mass, double dt,
                    bool both, hipStream_t s) {
    hipLaunchKernelGGL(kick_drift_kernel, dim3((unsigned)cdiv(n, KB)), dim3(KB), 0, s, n, pos, vel, force, mass,
                       0.5 * dt, dt, both ? 1 : 0);
    TFMM_LAUNCHED();
}

}  // namespace tfmm
