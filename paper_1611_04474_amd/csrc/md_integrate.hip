// Motion update around the force path: velocity Verlet (each MD iteration computes the
// forces on every atom, then updates the atoms' motion: Section 1, Section 2.1; the paper
// names no integrator). Positions, velocities and forces stay in HBM in the caller's order;
// one thread per atom. Units: A, fs, amu, kcal/mol.
#include "md_vv.hpp"

namespace md {
namespace {

// The first half kick and drift of a run: v += h a; x += dt v, wrapped. Later steps' are done by
// the step before (k_finalize_vv, k_vv_update), as are the second half kicks.
__global__ __launch_bounds__(256) void k_vv_kick_drift(int64_t n, float* __restrict__ pos,
                                                       float* __restrict__ vel,
                                                       const float* __restrict__ force,
                                                       const float* __restrict__ inv_mass,
                                                       float h, float dt, float L0, float L1,
                                                       float L2) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float s = inv_mass[i] * kAccel;
  const float L[3] = {L0, L1, L2};
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float v = fmaf(h * s, force[3 * i + c], vel[3 * i + c]);
    vel[3 * i + c] = v;
    pos[3 * i + c] = vv_drift(pos[3 * i + c], v, dt, L[c]);
  }
}

// vv_atom for every atom in the caller's order (larger systems, whose state is better streamed
// than visited in sorted order); block 0 adds the previous step's kinetic energies.
__global__ __launch_bounds__(256) void k_vv_update(int64_t n, const float* __restrict__ force,
                                                   VvArgs v) {
  if (blockIdx.x == 0) {
    if (v.ke_prev) ke_sum(v.kpart_prev, ke_blocks(n), v.ke_prev);
    return;
  }
  const int64_t i = ((int64_t)blockIdx.x - 1) * 256 + threadIdx.x;
  double e = 0.0;
  if (i < n) {
    const float f[3] = {force[3 * i], force[3 * i + 1], force[3 * i + 2]};
    e = vv_atom(v, i, vv_load(v, i), f);
  }
  e = block_sum(e);
  if (threadIdx.x == 0) v.kpart[blockIdx.x - 1] = e;
}

// the last step's kinetic energy
__global__ __launch_bounds__(kKeThreads) void k_ke_sum(const double* __restrict__ kpart,
                                                       int64_t nb, double* __restrict__ ke) {
  ke_sum(kpart, nb, ke);
}

}  // namespace

hipError_t launch_vv_kick_drift(int64_t n, float* pos, float* vel, const float* force,
                                const float* inv_mass, float h, float dt, const float* L,
                                hipStream_t stream) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_vv_kick_drift, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, n,
                     pos, vel, force, inv_mass, h, dt, L[0], L[1], L[2]);
  return hipGetLastError();
}

hipError_t launch_vv_update(int64_t n, const float* force, const VvArgs& v, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_vv_update, dim3((unsigned)ke_blocks(n) + 1), dim3(256), 0, stream, n, force, v);
  return hipGetLastError();
}

hipError_t launch_ke_sum(int64_t n, const double* kpart, double* ke, hipStream_t stream) {
  hipLaunchKernelGGL(k_ke_sum, dim3(1), dim3(kKeThreads), 0, stream, kpart, n > 0 ? ke_blocks(n) : 0,
                     ke);
  return hipGetLastError();
}

}  // namespace md
