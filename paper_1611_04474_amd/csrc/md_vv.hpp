// The motion update's arithmetic, shared by its own kernels (md_integrate.hip) and the force
// path's last kernel (md_finalize.hip).
#pragma once

#include "md_common.hpp"

namespace md {

constexpr float kAccel = 4.184e-4f;    // (kcal/mol/A)/amu in A/fs^2
constexpr int kKeThreads = 256;

// x + dt v, wrapped into [0, L) by one add or subtract of L (a step moves an atom far less
// than a box edge; one that moved farther stays outside and the force path flags it)
__device__ inline float vv_drift(float x, float v, float dt, float L) {
  x = fmaf(dt, v, x);
  if (x >= L) x -= L;
  else if (x < 0.f) x += L;
  return x;
}

// Atom i's velocity, position (where it is moved) and inverse mass.
struct VvState {
  struct F3 {
    float x[3];
  } v, x;
  float im;
};
__device__ inline VvState vv_load(const VvArgs& a, int64_t i) {
  VvState w;
  w.v = *reinterpret_cast<const VvState::F3*>(a.vel + 3 * i);
  if (a.drift) w.x = *reinterpret_cast<const VvState::F3*>(a.pos + 3 * i);
  w.im = a.inv_mass[i];
  return w;
}

// A step's second half kick by the force f and, with drift set, the next step's first half kick
// and drift. Returns the kinetic energy after the step, m v^2 / 2 in amu A^2/fs^2 (a pinned
// atom, 1/m = 0, has none).
__device__ inline double vv_atom(const VvArgs& a, int64_t i, VvState w, const float (&f)[3]) {
  const float hs = a.h * (w.im * kAccel);
  double v2 = 0.0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    w.v.x[c] = fmaf(hs, f[c], w.v.x[c]);
    v2 += (double)w.v.x[c] * (double)w.v.x[c];
    if (a.drift) {
      w.v.x[c] = fmaf(hs, f[c], w.v.x[c]);
      w.x.x[c] = vv_drift(w.x.x[c], w.v.x[c], a.dt, a.L[c]);
    }
  }
  *reinterpret_cast<VvState::F3*>(a.vel + 3 * i) = w.v;
  if (a.drift) *reinterpret_cast<VvState::F3*>(a.pos + 3 * i) = w.x;
  return w.im > 0.f ? 0.5 * v2 / (double)w.im : 0.0;
}

// Sum over a workgroup of 256 in a fixed order: within each wave, then the four waves.
__device__ inline double block_sum(double e) {
  __shared__ double s_e[kKeThreads / 64];
  for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off);
  if ((threadIdx.x & 63) == 0) s_e[threadIdx.x >> 6] = e;
  __syncthreads();
  return (s_e[0] + s_e[1]) + (s_e[2] + s_e[3]);
}

// The blocks' kinetic energies (amu A^2/fs^2) summed by one workgroup in a fixed order, in
// kcal/mol.
__device__ inline void ke_sum(const double* kpart, int64_t nb, double* ke) {
  double e = 0.0;
  for (int64_t b = threadIdx.x; b < nb; b += kKeThreads) e += kpart[b];
  e = block_sum(e);
  if (threadIdx.x == 0) *ke = e / (double)kAccel;
}

}  // namespace md
