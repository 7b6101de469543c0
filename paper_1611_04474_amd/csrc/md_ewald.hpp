// Shared by the two forms of the Ewald reciprocal-space sum (md_ewald.hip, md_ewald_mesh.hip).
#pragma once

#include "md_common.hpp"

namespace md {

// x as a fraction of the box edge L, 32-bit fixed point; st gets MD_STATUS_NAN for a NaN.
__device__ inline uint32_t ew_fraction(float xf, double L, uint32_t& st) {
  const double x = (double)xf;
  if (x != x) {
    st |= MD_STATUS_NAN;
    return 0;
  }
  const double s = x / L;
  const double f = s - floor(s);                                     // [0, 1)
  return (uint32_t)(unsigned long long)llrint(f * 4294967296.0);     // 2^32 wraps to 0
}

// Atom i's fractions and its charge's bits.
__device__ inline uint4 ew_fractions(const float* pos, const float* q, const double* L, int64_t i,
                                     uint32_t& st) {
  uint4 u;
  u.x = ew_fraction(pos[3 * i + 0], L[0], st);
  u.y = ew_fraction(pos[3 * i + 1], L[1], st);
  u.z = ew_fraction(pos[3 * i + 2], L[2], st);
  const float qi = q[i];
  if (qi != qi) st |= MD_STATUS_NAN;
  u.w = __float_as_uint(qi);
  return u;
}

// One workgroup of 256: energy partials, then self and background terms, in a fixed order.
__device__ inline void ew_energy_sum(const double* epart, int64_t ne, const double2* qpart,
                                     int64_t nq, const double* L, double alpha, double coulomb_k,
                                     double* energy) {
  __shared__ double s[256], s2[256], s1[256];
  double e = 0.0, q2 = 0.0, q1 = 0.0;
  for (int64_t t = threadIdx.x; t < ne; t += 256) e += epart[t];
  for (int64_t t = threadIdx.x; t < nq; t += 256) {
    q2 += qpart[t].x;
    q1 += qpart[t].y;
  }
  s[threadIdx.x] = e;
  s2[threadIdx.x] = q2;
  s1[threadIdx.x] = q1;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) {
      s[threadIdx.x] += s[threadIdx.x + off];
      s2[threadIdx.x] += s2[threadIdx.x + off];
      s1[threadIdx.x] += s1[threadIdx.x + off];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double pi = 3.141592653589793;
    const double V = L[0] * L[1] * L[2];
    const double self = -coulomb_k * alpha / sqrt(pi) * s2[0];
    const double bg = -coulomb_k * pi * s1[0] * s1[0] / (2.0 * V * alpha * alpha);
    *energy = s[0] + self + bg;
  }
}

// Grid form (md_ewald_mesh.hip).
struct EwMeshPlan {
  int K[3], N[3], M[3], nt[3];  // kmax; basis functions (2 (K + 1) up to a multiple of 16); grid
                                // points; tiles
  int64_t nbins, nepart, qblocks;
  size_t off_ups, off_rec, off_win, off_dwin, off_slot, off_ids, off_sid, off_count, off_start,
      off_buf0, off_buf1, off_buf2, off_pot, off_tab[3], off_tabT[3], off_gfac[3], off_ksq[3],
      off_epart, off_qpart, total;
};

struct EwMeshArgs {
  int64_t n;
  const float* pos;    // [n][3], caller order
  const float* q;      // [n]
  float* force;        // [n][3]
  double* energy;      // [1]
  int accumulate;
  WsHeader* hdr;
  uint4* ups;          // [n] fractions and charge, caller order
  uint4* rec;          // [n] the same by bin, in index order within a bin
  float *win, *dwin;   // [n][32] by bin: window values and derivatives, 10 per axis, x
                       // (times the charge), y, z
  int2* slot;          // [n] bin and place in it
  int* ids;            // [n] indices by bin
  int* sid;            // [n] indices by bin, in order
  int* count;          // [nbins], pad words apart
  int* start;          // [nbins + 1]
  float* buf0;         // [Mx][My][Mz] charges
  double* pot;         // [Mx][My][Mz] the potential's coefficients, in the same place
  float* buf1;         // [Mx][Ny][Nz] charges transformed along z and y
  double* buf2;        // the same of the potential, transformed back along x
  double *tab[3], *tabT[3];  // [N][M] and [M][N] basis functions per axis
  double *gfac[3], *ksq[3];  // [N] per axis: multiplicity exp(-k^2/4 alpha^2)/phihat^2; k^2
  double* epart;       // [nepart]
  double2* qpart;      // [qblocks] sum q^2, sum q
  int64_t nepart, qblocks, nbins;
  int pad;
  int M[3], N[3], K[3], nt[3];
  double cb[3];        // the windows' shape: beta log2(e)
  double L[3], mL[3], alpha, coulomb_k, gscale;   // mL = M / L
};

// The grid form takes systems of at least so many atoms with these wave numbers.
int64_t ew_mesh_from(const int32_t kmax[3]);
void ew_mesh_plan(int64_t n, const int32_t kmax[3], EwMeshPlan* pl);
hipError_t launch_ew_mesh(const EwMeshPlan& pl, const md_params* p, int64_t n, const float* pos,
                          const float* q, float* force, double* energy, int accumulate, void* ws,
                          hipStream_t st);

}  // namespace md
