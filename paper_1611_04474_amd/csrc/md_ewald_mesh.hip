// Ewald reciprocal-space sum of larger systems: the same sum over wave vectors as
// md_ewald.hip, through a non-uniform Fourier transform, O(N + grid) instead of O(N K).
//
// The charges are spread to a regular grid with a window wide enough that the gridding error
// (3e-8 of the forces at an oversampling of 1.75, from a float64 comparison with the direct
// sum) lies below float32 rounding, so this is not a particle-mesh approximation with an
// accuracy to choose: forces and energy are no further from a float64 sum than the direct sum's
// (see the accuracy at ew_mesh_from). With real separable basis functions t_n(l), n = 2 m + a:
// cos (a = 0) or sin (a = 1) of 2 pi m l / M, the pieces are
//   b[l]    = sum_j q_j phi(l_x - X_j) phi(l_y - Y_j) phi(l_z - Z_j),   X = M_x u_x, ...
//   R[n]    = sum_l b[l] t_nx(l_x) t_ny(l_y) t_nz(l_z)
//   Q[n]    = (4 pi k / V) mu(m) exp(-|kv|^2/(4 alpha^2)) / |kv|^2 / phihat(m)^2  R[n]
//   E       = 1/2 sum_n Q[n] R[n]
//   c[l]    = sum_n Q[n] t_nx t_ny t_nz
//   F_j     = q_j sum_l c[l] (M_x/L_x phi'(l_x - X_j) phi phi, ...)
// with mu the number of distinct sign choices of the mode m >= 0 (the characters of the sign
// flips are orthogonal, so the sum over +-m of |S|^2 is mu times the sum of the squares of
// R over the eight cos/sin choices, and the potential has the coefficients mu R), and phihat
// the window's transform. The window is phi(t) = exp(beta (sqrt(1 - (2t/w)^2) - 1)) on
// |t| < w/2, w = 10 grid points (Barnett, Magland and af Klinteberg, SIAM J. Sci. Comput. 41
// (2019) C479), with beta from the axis's oversampling.
//
// Grids have a few million points at most and only the modes |m| <= kmax are wanted, so the
// transforms are products with a table of sines and cosines per axis on the matrix cores
// (float64 MFMA), any grid size, a few GFLOP; a fast Fourier transform would save operations
// that are not the bound. Kernels:
//   k_em_init     tables, window transforms, counters
//   k_em_setup    per atom: fractions, NaN check, partial sums of q^2 and q; bin count
//   k_em_place    bin starts and atom indices to bins; many bins: k_em_scan, k_em_scatter
//   k_em_sort     each bin in index order (so sums run in a fixed order)
//   k_em_spread   b, one workgroup per tile of 8 x 8 x 16 grid points
//   k_em_forward, k_em_middle, k_em_back   the axis transforms z y, x (Q and E) x, y z
//   k_em_force    forces, one workgroup per tile
//   k_em_energy   fixed-order sum of the energy partials, self and background
// Every sum runs in a fixed order: the results are the same bits on every run.
#include <math.h>

#include "md_ewald.hpp"

namespace md {
namespace {

constexpr int kW = 10;                  // window width in grid points
constexpr int kTX = 8, kTZ = 16;        // tile: 8 x 8 x 16 grid points
constexpr int kLo = kW / 2 - 1;         // an atom at grid cell l covers l - 4 .. l + 5
constexpr int kHi = kW / 2;
// Grids of at most kPlaceBins bins (EwMeshArgs::pad): the bin counters lie 32 bytes apart, so
// that atomics of neighbouring bins do not wait for each other's line (k_em_setup of 92,224
// atoms in 2,268 bins 13.2 -> 7.4 us; 128 bytes apart 6.6). With more bins the atomics spread
// by themselves, and one workgroup scans the counts (100,000 atoms in 32,000 bins, whole sum:
// 1142 us apart, 1128 packed).
constexpr int kPad = 8, kPlaceBins = 4096;
inline int64_t mesh_pad(int64_t nbins) { return nbins <= kPlaceBins ? kPad : 1; }
typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));

// The window phi(t) = exp(beta (sqrt(1 - x^2) - 1)), x = 2 t / w, and its derivative, for
// t = r - f with r a whole number of grid points and f a 32-bit fraction (both exact); c =
// beta log2(e). Formed in float64 and rounded once (the reciprocal root from a float32 one and a
// Newton step, 2^h by the exponential series to h^8, 2e-10): the hardware's 2^x is a little low on
// average, 2e-8 of the energy and 3e-8 of the forces over three axes (k_em_sort, which forms the
// windows, 12.8 us with it, 14.0 without). In float32 throughout the exponent's
// rounding alone put 3e-7 into the forces.
__device__ inline float window(int r, uint32_t f, double c, float& d) {
  const double t = fma((double)f, -2.3283064365386963e-10, (double)r);   // 2^-32
  const double x = t * (2.0 / kW);
  const double y = fma(-x, x, 1.0);
  const float rs = __builtin_amdgcn_rsqf(fmaxf((float)y, 1e-7f));
  const double r0 = (double)rs;
  const double ri = fma(0.5 * r0, fma(-y * r0, r0, 1.0), r0);   // 1/sqrt(y)
  const double g = c * fma(y, ri, -1.0);
  const double k = rint(g), h = (g - k) * 0.6931471805599453;
  double e = 1.0 / 40320.0;
  e = fma(e, h, 1.0 / 5040.0);
  e = fma(e, h, 1.0 / 720.0);
  e = fma(e, h, 1.0 / 120.0);
  e = fma(e, h, 1.0 / 24.0);
  e = fma(e, h, 1.0 / 6.0);
  e = fma(e, h, 0.5);
  e = fma(e, h, 1.0);
  e = fma(e, h, 1.0);
  e = y > 1e-7 ? __builtin_amdgcn_ldexp(e, (int)k) : 0.0;
  d = (float)(e * (-x * (c * (0.6931471805599453 * 2.0 / kW))) * ri);
  return (float)e;
}

// Grid cell of a 32-bit fraction u on an axis of M points; f: the offset within it as a 32-bit
// fraction.
__device__ inline int grid_cell(uint32_t u, int M, uint32_t& f) {
  const uint64_t p = (uint64_t)u * (uint32_t)M;
  f = (uint32_t)p;
  return (int)(p >> 32);
}

__device__ inline int bin_of(const EwMeshArgs& a, uint4 u) {
  uint32_t f;
  const int x = grid_cell(u.x, a.M[0], f) / kTX, y = grid_cell(u.y, a.M[1], f) / kTX,
            z = grid_cell(u.z, a.M[2], f) / kTZ;
  return (x * a.nt[1] + y) * a.nt[2] + z;
}

// Blocks 0 .. nb_tab - 1: the tables, an entry per thread; then one wave per (axis, mode):
// the window's transform by the trapezoid rule (its integrand is smooth to e^-beta at the
// ends, so 320 points leave no error in float64) and the mode's factors; the bin counters are
// cleared by every block.
__global__ __launch_bounds__(256) void k_em_init(EwMeshArgs a, unsigned nb_tab) {
  const int64_t gt = (int64_t)blockIdx.x * 256 + threadIdx.x;
  for (int64_t i = gt; i < a.pad * a.nbins; i += (int64_t)gridDim.x * 256) a.count[i] = 0;
  if (gt == 0) a.hdr->status = 0;
  if (blockIdx.x < nb_tab) {
    int64_t e = gt;
    for (int d = 0; d < 3; ++d) {
      const int64_t sz = (int64_t)a.N[d] * a.M[d];
      if (e < sz) {
        const int n = (int)(e / a.M[d]), l = (int)(e % a.M[d]);
        const int m = n >> 1;
        double s = 0.0, c = 0.0;
        if (m <= a.K[d]) sincospi(2.0 * (double)(((int64_t)m * l) % a.M[d]) / (double)a.M[d], &s, &c);
        const double v = (n & 1) ? s : c;
        a.tab[d][e] = v;                                   // [n][l]
        a.tabT[d][(int64_t)l * a.N[d] + n] = v;            // [l][n]
        return;
      }
      e -= sz;
    }
    return;
  }
  const int wv = (int)(blockIdx.x - nb_tab) * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  int m = wv, d = 0;
  while (d < 3 && m >= a.N[d] / 2) {
    m -= a.N[d] / 2;
    ++d;
  }
  if (d >= 3) return;
  double sum = 0.0;
  const double xi = (double)m / (double)a.M[d];
  for (int p = lane; p < 160; p += 64) {
    const double t = ((double)p + 0.5) / 32.0;             // 0 .. 5, the even half
    const double x = t * (2.0 / kW);
    sum += exp2(a.cb[d] * (sqrt(1.0 - x * x) - 1.0)) * cospi(2.0 * xi * t);
  }
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if (lane != 0) return;
  const double ph = sum / 16.0;                            // 2 h sum, h = 1/32
  const double k = 2.0 * M_PI * (double)m / a.L[d];
  const double g = m <= a.K[d] ? (m > 0 ? 2.0 : 1.0) * exp(-k * k / (4.0 * a.alpha * a.alpha)) / (ph * ph)
                               : 0.0;
  a.gfac[d][2 * m] = a.gfac[d][2 * m + 1] = g;
  a.ksq[d][2 * m] = a.ksq[d][2 * m + 1] = k * k;
}

__global__ __launch_bounds__(256) void k_em_setup(EwMeshArgs a) {
  __shared__ double s_q2[4], s_q1[4];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  double q2 = 0.0, q1 = 0.0;
  int b = 0, at = 0;
  if (i < a.n) {
    uint32_t st = 0;
    const uint4 u = ew_fractions(a.pos, a.q, a.L, i, st);
    b = bin_of(a, u);
    at = atomicAdd(&a.count[(int64_t)a.pad * b], 1);   // on its way during the sums below
    a.ups[i] = u;
    const double qi = (double)__uint_as_float(u.w);
    q2 = qi * qi;
    q1 = qi;
    if (st) atomicOr(&a.hdr->status, st);
  }
  for (int off = 32; off > 0; off >>= 1) {
    q2 += __shfl_xor(q2, off);
    q1 += __shfl_xor(q1, off);
  }
  if ((threadIdx.x & 63) == 0) {
    s_q2[threadIdx.x >> 6] = q2;
    s_q1[threadIdx.x >> 6] = q1;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    a.qpart[blockIdx.x] = make_double2((s_q2[0] + s_q2[1]) + (s_q2[2] + s_q2[3]),
                                       (s_q1[0] + s_q1[1]) + (s_q1[2] + s_q1[3]));
  if (i < a.n) a.slot[i] = make_int2(b, at);
}

// Exclusive scan of the bin counts, one workgroup, 4 bins per thread and round.
__global__ __launch_bounds__(1024) void k_em_scan(EwMeshArgs a) {
  __shared__ int s_w[16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  int carry = 0;
  for (int64_t b0 = 0; b0 < a.nbins; b0 += 4096) {
    int v[4], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t b = b0 + 4 * t + k;
      v[k] = b < a.nbins ? a.count[b] : 0;
      sum += v[k];
    }
    int inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(inc, o);
      if (lane >= o) inc += y;
    }
    if (lane == 63) s_w[w] = inc;
    __syncthreads();
    int before = carry, all = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      before += k < w ? s_w[k] : 0;
      all += s_w[k];
    }
    __syncthreads();
    int ex = before + inc - sum;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t b = b0 + 4 * t + k;
      if (b < a.nbins) a.start[b] = ex;
      ex += v[k];
    }
    carry += all;
  }
  if (t == 0) a.start[a.nbins] = carry;
}

__global__ __launch_bounds__(256) void k_em_scatter(EwMeshArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.n) return;
  const int2 s = a.slot[i];
  a.ids[a.start[s.x] + s.y] = (int)i;
}

// Grids of at most kPlaceBins bins: every block scans the counts itself and then places its atoms,
// which costs less than the launch of a scan between (92,224 atoms in 2,268 bins: 9.5 us for
// both, 5.4 this way; the reciprocal call 151.5 -> 149.9). Block 0 writes the starts.
constexpr int kPlaceThreads = 1024;
__global__ __launch_bounds__(kPlaceThreads) void k_em_place(EwMeshArgs a) {
  constexpr int kPer = kPlaceBins / kPlaceThreads, kNW = kPlaceThreads / 64;
  __shared__ int s_start[kPlaceBins], s_w[kNW];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, nb = (int)a.nbins;
  const int64_t i = (int64_t)blockIdx.x * kPlaceThreads + t;
  const int2 s = i < a.n ? a.slot[i] : make_int2(0, 0);
  int v[kPer], sum = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int b = kPer * t + k;
    v[k] = b < nb ? a.count[kPad * b] : 0;
    sum += v[k];
  }
  int inc = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  if (lane == 63) s_w[w] = inc;
  __syncthreads();
  int ex = inc - sum;
#pragma unroll
  for (int k = 0; k < kNW; ++k) ex += k < w ? s_w[k] : 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int b = kPer * t + k;
    s_start[b] = ex;
    if (blockIdx.x == 0 && b < nb) a.start[b] = ex;
    ex += v[k];
  }
  if (blockIdx.x == 0 && t == 0) a.start[nb] = (int)a.n;
  __syncthreads();
  if (i < a.n) a.ids[s_start[s.x] + s.y] = (int)i;
}

// One workgroup per bin: its atoms in index order, so that the spreading adds in a fixed order.
// Up to kRankMax members rank by counting smaller indices; a fuller bin marks them in a bit
// map of kMapBits consecutive indices at a time and lists the marked ones. Then the atoms'
// window values and derivatives, 10 per axis, half a wave per atom, those of x times the charge:
// the spreading, which meets an atom in about 7 tiles, and the forces read them back.
constexpr int kRankMax = 256, kMapBits = 32768;
__global__ __launch_bounds__(256) void k_em_sort(EwMeshArgs a) {
  __shared__ uint32_t s_map[kMapBits / 32];
  __shared__ uint4 s_rec[kRankMax];
  __shared__ int s_w[4];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t b = blockIdx.x;
  const int s = a.start[b], m = a.start[b + 1] - s;
  if (m == 0) return;
  const bool small = m <= kRankMax;
  if (small) {
    const int id = t < m ? a.ids[s + t] : 0x7fffffff;
    const uint4 u = t < m ? a.ups[id] : make_uint4(0, 0, 0, 0);
    s_map[t] = (uint32_t)id;
    __syncthreads();
    int rank = 0;
    if (t < m)
      for (int j = 0; j < m; ++j) rank += (int)s_map[j] < id ? 1 : 0;
    if (t < m) {
      a.rec[s + rank] = u;
      s_rec[rank] = u;
      a.sid[s + rank] = id;
    }
  } else {
    int out = s;
    for (int64_t i0 = 0; i0 < a.n; i0 += kMapBits) {
      for (int e = t; e < kMapBits / 32; e += 256) s_map[e] = 0;
      __syncthreads();
      for (int e = t; e < m; e += 256) {
        const int64_t r = (int64_t)a.ids[s + e] - i0;
        if (r >= 0 && r < kMapBits) atomicOr(&s_map[r >> 5], 1u << (r & 31));
      }
      __syncthreads();
      for (int e0 = 0; e0 < kMapBits / 32; e0 += 256) {
        uint32_t v = s_map[e0 + t];
        const int c = __builtin_popcount(v);
        int inc = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int y = __shfl_up(inc, o);
          if (lane >= o) inc += y;
        }
        if (lane == 63) s_w[w] = inc;
        __syncthreads();
        int p = out + inc - c;
        for (int k = 0; k < 4; ++k) {
          p += k < w ? s_w[k] : 0;
          out += s_w[k];
        }
        while (v) {
          const int i = (int)(i0 + 32 * (e0 + t) + __builtin_ctz(v));
          a.rec[p] = a.ups[i];
          a.sid[p] = i;
          ++p;
          v &= v - 1;
        }
        __syncthreads();   // s_w and the map are used again
      }
    }
    __threadfence_block();   // the records are read back
  }
  __syncthreads();
  const int c = lane & 31, d = min(c / kW, 2), k = c % kW;
  const double cb = a.cb[d];
  const int M = a.M[d];
  for (int e = t >> 5; e < m; e += 8) {
    const uint4 u = small ? s_rec[e] : a.rec[s + e];
    uint32_t f;
    grid_cell(d == 0 ? u.x : d == 1 ? u.y : u.z, M, f);
    float dw;
    float v = window(k - kLo, f, cb, dw);
    if (d == 0) {
      v *= __uint_as_float(u.w);
      dw *= __uint_as_float(u.w);
    }
    if (c < 3 * kW) {
      a.win[(int64_t)(s + e) * 32 + c] = v;
      a.dwin[(int64_t)(s + e) * 32 + c] = dw;
    }
  }
}

// The charges' grid, one workgroup of 4 waves per tile of 8 x 8 x 16 points: as a matrix
// product over the atoms near the tile, b[(x, y)][z] = sum_j (q phi_x phi_y)[(x, y)][j]
// phi_z[j][z], on the matrix cores, wave w taking x = 2 w and 2 w + 1. The atoms come from
// the tile's own bin and the 26 around it (each axis has at least three), wave w looking
// through bins w, w + 4, ..; those whose window meets the tile (one in four) go to the wave's
// list, and their windows are laid out over the tile's points kSub atoms at a time. In a
// 16x16x4 f32 product lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and holds
// D[4 (l / 16) + i][l % 16].
constexpr int kList = 256, kSub = 64, kNear = 27;
__global__ __launch_bounds__(256) void k_em_spread(EwMeshArgs a) {
  __shared__ int s_start[28], s_cnt[28];
  __shared__ int s_at[4][kList], s_rel[4][kList];   // sorted position; x, y, z + 8 off the tile
  __shared__ float s_w[kSub][32 + 2];         // per atom: 8 x, 8 y and 16 z points of the tile
  __shared__ int s_n[4], s_more;
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const int tz = blockIdx.x % a.nt[2], ty = (blockIdx.x / a.nt[2]) % a.nt[1],
            tx = blockIdx.x / (a.nt[2] * a.nt[1]);
  if (t < 28) {
    int bx = tx + t / 9 - 1, by = ty + (t / 3) % 3 - 1, bz = tz + t % 3 - 1;
    bx += bx < 0 ? a.nt[0] : bx >= a.nt[0] ? -a.nt[0] : 0;
    by += by < 0 ? a.nt[1] : by >= a.nt[1] ? -a.nt[1] : 0;
    bz += bz < 0 ? a.nt[2] : bz >= a.nt[2] ? -a.nt[2] : 0;
    const int b = t < kNear ? (bx * a.nt[1] + by) * a.nt[2] + bz : 0;
    s_start[t] = a.start[b];
    s_cnt[t] = t < kNear ? a.start[b + 1] - s_start[t] : 0;
  }
  __syncthreads();
  v4f acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
  const int row = lane & 15, kk = lane >> 4;
  // the first 64 atoms of this wave's bins, all loads in flight
  constexpr int kBins = (kNear + 3) / 4;
  uint4 u[kBins];
#pragma unroll
  for (int k = 0; k < kBins; ++k) {
    const int b = 4 * k + w;   // at most 27, which is empty
    u[k] = a.rec[lane < s_cnt[b] ? s_start[b] + lane : 0];
  }
  int n = 0;   // atoms listed by this wave
  auto list = [&](int b, int e0, const uint4& v) {
    const int e = e0 + lane;
    const int dx = b / 9 - 1, dy = (b / 3) % 3 - 1, dz = b % 3 - 1;
    // the grid cell relative to the tile: within the bin, and the bin's own offset
    const int rx = (int)(__umulhi(v.x, (uint32_t)a.M[0]) % kTX) + kTX * dx;
    const int ry = (int)(__umulhi(v.y, (uint32_t)a.M[1]) % kTX) + kTX * dy;
    const int rz = (int)(__umulhi(v.z, (uint32_t)a.M[2]) % kTZ) + kTZ * dz;
    const bool keep = e < s_cnt[b] && rx >= -kHi && rx < kTX + kLo && ry >= -kHi &&
                      ry < kTX + kLo && rz >= -kHi && rz < kTZ + kLo;
    const unsigned long long m = __builtin_amdgcn_ballot_w64(keep);
    if (keep) {
      const int at = n + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
      s_at[w][at] = s_start[b] + e;
      s_rel[w][at] = (rx + 8) | (ry + 8) << 8 | (rz + 8) << 16;
    }
    n += __builtin_popcountll(m);
  };
  // next atom to look at: bin kb, from e; a list has room for 64 more before each step
  int kb = 0, eb = 0;
  bool first = true;
  for (;;) {
    if (first) {
#pragma unroll
      for (int k = 0; k < kBins; ++k) {
        if (n <= kList - 64 && kb == k && eb == 0) {
          const int b = 4 * k + w;
          if (s_cnt[b] > 0) list(b, 0, u[k]);
          if (s_cnt[b] > 64) eb = 64;   // the rest of a fuller bin below
          else ++kb;
        }
      }
    }
    while (kb < kBins && n <= kList - 64) {
      const int b = 4 * kb + w;
      if (eb < s_cnt[b]) {
        list(b, eb, a.rec[s_start[b] + min(eb + lane, s_cnt[b] - 1)]);
        eb += 64;
      } else {
        ++kb;
        eb = 0;
      }
    }
    first = false;
    if (t == 0) s_more = 0;
    if (lane == 0) s_n[w] = n;
    __syncthreads();
    if (lane == 0 && kb < kBins) s_more = 1;
    const int n0 = s_n[0], n1 = n0 + s_n[1], n2 = n1 + s_n[2], tot = n2 + s_n[3];
    // window values at the tile's points, 32 per atom (past the last atom zeros), those of the
    // next kSub atoms on their way while the matrix cores take the last ones
    constexpr int kVals = 32 * kSub / 256;
    float val[kVals];
    auto fetch = [&](int j0) {
      const int c = t & 31;
      const int off = c < 8 ? 0 : c < 16 ? kW : 2 * kW, sh = c < 8 ? 0 : c < 16 ? 8 : 16;
      const int x = (c < 8 ? c : c < 16 ? c - 8 : c - 16) + kLo + 8;
#pragma unroll
      for (int k = 0; k < kVals; ++k) {
        const int j = j0 + 8 * k + (t >> 5);
        val[k] = 0.f;
        if (j < tot) {
          const int v = (j >= n0) + (j >= n1) + (j >= n2);
          const int jj = j - (v == 0 ? 0 : v == 1 ? n0 : v == 2 ? n1 : n2);
          const int i = x - ((s_rel[v][jj] >> sh) & 255);   // the window's point
          if (i >= 0 && i < kW) val[k] = a.win[(int64_t)s_at[v][jj] * 32 + (off + i)];
        }
      }
    };
    if (tot > 0) fetch(0);
    for (int j0 = 0; j0 < tot; j0 += kSub) {
      const int n8 = (min(kSub, tot - j0) + 7) & ~7;
#pragma unroll
      for (int k = 0; k < kVals; ++k) s_w[8 * k + (t >> 5)][t & 31] = val[k];
      __syncthreads();
      if (j0 + kSub < tot) fetch(j0 + kSub);
      for (int s = 0; s < n8; s += 8) {
        const float *wa = s_w[s + kk], *wb = s_w[s + 4 + kk];
        const float va = wa[2 * w + (row >> 3)] * wa[8 + (row & 7)];
        const float vb = wb[2 * w + (row >> 3)] * wb[8 + (row & 7)];
        acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(va, wa[16 + row], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(vb, wb[16 + row], acc1, 0, 0, 0);
      }
      __syncthreads();
    }
    __syncthreads();   // s_more is set, the lists are read
    if (!s_more) break;
    n = 0;
    __syncthreads();   // before s_more is cleared
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int p = 16 * w + 4 * kk + i;
    const int64_t x = kTX * tx + (p >> 3), y = kTX * ty + (p & 7);
    a.buf0[(x * a.M[1] + y) * a.M[2] + kTZ * tz + row] = acc0[i] + acc1[i];
  }
}

// Axis transforms, on the matrix cores in float64. With float32 products, summed in float64 by
// groups of 16, the rounding of a group left noise of a grid point's width in the potential, which the
// derivative multiplies by the points per wavelength, and float32 tables put 7e-8 into the energy;
// the potential's intermediates are kept in float64 too, since noise along one axis alone counts
// four times that of the stored grid, which the window averages over the other two, and so is the
// stored grid, whose rounding follows the longest waves of the box. RMS force error, float32 products, float64
// ones, float64 intermediates, and grid: 92,224 atoms 4.4e-7, 1.4e-7, 8.4e-8, 7.7e-8; 9,001 with twice
// the wave numbers they need 5.9e-7, 1.8e-7, 9.4e-8, 7.8e-8; 33,880 in a 22 x 22 x 700 A box
// 5.8e-7 with float64 intermediates, 8.9e-8 with the grid.
// A lane's latency to memory, not the products (1.2 GFLOP, 15 us for all
// six at 92,224 atoms), is what a transform takes its time for, so each kernel does two of them: z
// and y of a plane, x forward and back of a column, y and z of a plane, the intermediate in LDS.
// 92,224 atoms (grid 144 x 144 x 112, 80 x 80 x 64 modes): 60.1 us in six launches of
// float32 products, 43.2 in these three, 61.5 in float64.
constexpr int kTrWaves = 8, kTrThreads = 64 * kTrWaves;

// (p + a 32-bit byte offset: one uniform base and a lane offset per load)
template <typename T>
__device__ inline T word_at(const T* p, uint32_t byte) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + byte);
}

// 16 rows x 16 C columns, sum over K: step s of a group of 16 k uses k0 + 4 (l / 16) + s for both
// sides; fa(k) gives a lane its row's four consecutive k (a float4 or double4), fb(k, v) the columns of
// them. Each of A (rows) and two (columns) groups' operands has registers of its own and is loaded
// again as soon as it is used, so the loads of the following groups are always on their way. In a
// 16x16x4 f64 product lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and holds
// D[l / 16 + 4 i][l % 16].
template <int C, int A, typename FA, typename FB>
__device__ __attribute__((always_inline)) inline void rows_times(int K, FA fa, FB fb, v4d (&acc)[C]) {
  decltype(fa(0)) av[A];
  double bv[2][4][C];
#pragma unroll
  for (int g = 0; g < A; ++g) av[g] = fa(min(16 * g, K - 16));
#pragma unroll
  for (int g = 0; g < 2; ++g) fb(min(16 * g, K - 16), bv[g]);
  auto step = [&](int g, int k) __attribute__((always_inline)) {
    const double a4[4] = {(double)av[g % A].x, (double)av[g % A].y, (double)av[g % A].z, (double)av[g % A].w};
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int c = 0; c < C; ++c)
        acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a4[s], bv[g & 1][s][c], acc[c], 0, 0, 0);
    av[g % A] = fa(min(k + 16 * A, K - 16));
    fb(min(k + 32, K - 16), bv[g & 1]);
  };
  int k0 = 0;
  for (; k0 + 64 <= K; k0 += 64) {
#pragma unroll
    for (int g = 0; g < 4; ++g) step(g, k0 + 16 * g);
  }
#pragma unroll
  for (int g = 0; g < 3; ++g)
    if (k0 + 16 * g < K) step(g, k0 + 16 * g);
}

// 16 rows x 16 columns, sum over K: step s of a group uses k0 + 4 s + l / 16; fa(k, s), fb(k, s)
// give a lane its element of row and column k + 4 s. Operands of four groups on their way.
template <typename FA, typename FB>
__device__ __attribute__((always_inline)) inline void tile_times(int K, FA fa, FB fb, v4d& acc) {
  typedef decltype(fa(0, 0)) TA;
  typedef decltype(fb(0, 0)) TB;
  TA av[4][4];
  TB bv[4][4];
  auto load = [&](int k, TA (&va)[4], TB (&vb)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      va[s] = fa(k, s);
      vb[s] = fb(k, s);
    }
  };
#pragma unroll
  for (int g = 0; g < 4; ++g) load(min(16 * g, K - 16), av[g], bv[g]);
  auto step = [&](int g, int k, bool more) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)av[g][s], (double)bv[g][s], acc, 0, 0, 0);
    if (more) load(min(k + 64, K - 16), av[g], bv[g]);
  };
  int k0 = 0;
  for (; k0 + 64 <= K; k0 += 64) {
#pragma unroll
    for (int g = 0; g < 4; ++g) step(g, k0 + 16 * g, true);
  }
#pragma unroll
  for (int g = 0; g < 3; ++g)
    if (k0 + 16 * g < K) step(g, k0 + 16 * g, false);
}

// z and y forward: workgroup (x, group of up to C 16-column tiles of nz). The row stride in LDS
// is an odd number of 16s, so that the four k that a wave reads at once lie in different banks.
template <int C>
__global__ __launch_bounds__(kTrThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_em_forward(EwMeshArgs a, int groups) {
  extern __shared__ __attribute__((aligned(16))) float s_m[];   // [M1][16 (C | 1)]
  constexpr int kStride = 16 * (C | 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int row = lane & 15, kk = lane >> 4;
  const int64_t x = blockIdx.x / groups;
  const int M1 = a.M[1], M2 = a.M[2], N1 = a.N[1], N2 = a.N[2];
  const int c0 = (int)(blockIdx.x % groups) * C, nc = min(C, N2 / 16 - c0);
  for (int r = w; r < M1 / 16; r += kTrWaves) {
    const float* ip = a.buf0 + (x * M1 + 16 * r) * M2;
    const double* tp = a.tabT[2] + 16 * c0;
    const uint32_t io = 4 * (row * M2 + 4 * kk), to = 8 * (4 * kk * N2 + row);
    v4d acc[C] = {};
    rows_times<C, 4>(M2, [&](int k) { return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(ip) + (4u * k + io)); },
                  [&](int k, double (&v)[4][C]) {
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                      for (int c = 0; c < C; ++c) v[s][c] = word_at(tp, 8u * ((k + s) * N2 + 16 * min(c, nc - 1)) + to);
                  }, acc);
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) s_m[(16 * r + kk + 4 * i) * kStride + 16 * c + row] = (float)acc[c][i];
  }
  __syncthreads();
  for (int t = w; t < N1 / 16 * nc; t += kTrWaves) {
    const int i0 = t / nc * 16, c = t % nc;
    const double* tp = a.tabT[1] + i0;
    const uint32_t to = 8 * (kk * N1 + row);
    const float* bp = s_m + kk * kStride + 16 * c + row;
    v4d acc = {};
    tile_times(M1, [&](int k, int s) { return word_at(tp, 8u * (k + 4 * s) * N1 + to); },
               [&](int k, int s) { return bp[(k + 4 * s) * kStride]; }, acc);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      a.buf1[(x * N1 + i0 + kk + 4 * i) * N2 + 16 * (c0 + c) + row] = (float)acc[i];
  }
}

// x forward, the scaling of R to Q in float64 with the energy 1/2 sum Q R (a part per 16 x 16
// tile), and x back: workgroup j of 16 columns (ny, nz).
__global__ __launch_bounds__(kTrThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_em_middle(EwMeshArgs a) {
  extern __shared__ __attribute__((aligned(16))) float s_q[];   // [N0][16]
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int row = lane & 15, kk = lane >> 4;
  const int M0 = a.M[0], N0 = a.N[0];
  const int64_t J = (int64_t)a.N[1] * a.N[2], j = (int64_t)blockIdx.x * 16 + row;
  const int ny = (int)(j / a.N[2]), nz = (int)(j % a.N[2]);
  const double k2yz = a.ksq[1][ny] + a.ksq[2][nz];
  for (int t = w; t < N0 / 16; t += kTrWaves) {
    const double* tp = a.tabT[0] + 16 * t;
    const float* ip = a.buf1 + (int64_t)blockIdx.x * 16;
    const uint32_t to = 8 * (kk * N0 + row), io = 4 * (kk * (uint32_t)J + row);
    v4d acc = {};
    tile_times(M0, [&](int k, int s) { return word_at(tp, 8u * (k + 4 * s) * N0 + to); },
               [&](int k, int s) { return word_at(ip, 4u * (k + 4 * s) * (uint32_t)J + io); }, acc);
    double e = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int nx = 16 * t + kk + 4 * i;
      const double k2 = a.ksq[0][nx] + k2yz;
      const double g = k2 > 0.0 ? a.gscale * a.gfac[0][nx] * a.gfac[1][ny] * a.gfac[2][nz] / k2 : 0.0;
      const double q = g * acc[i];
      e += 0.5 * q * acc[i];
      s_q[nx * 16 + row] = (float)q;
    }
    for (int o = 32; o > 0; o >>= 1) e += __shfl_xor(e, o);
    if (lane == 0) a.epart[(int64_t)blockIdx.x * (N0 / 16) + t] = e;
  }
  __syncthreads();
  for (int t = w; t < M0 / 16; t += kTrWaves) {
    const double* tp = a.tab[0] + 16 * t;
    const uint32_t to = 8 * (kk * M0 + row);
    const float* bp = s_q + kk * 16 + row;
    v4d acc = {};
    tile_times(N0, [&](int k, int s) { return word_at(tp, 8u * (k + 4 * s) * M0 + to); },
               [&](int k, int s) { return bp[(k + 4 * s) * 16]; }, acc);
#pragma unroll
    for (int i = 0; i < 4; ++i) a.buf2[(16 * t + kk + 4 * i) * J + j] = acc[i];
  }
}

// y and z back: workgroup (x, group of up to rt 16-row tiles of y).
__global__ __launch_bounds__(kTrThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_em_back(EwMeshArgs a, int rt, int groups) {
  extern __shared__ __attribute__((aligned(16))) double s_r[];   // [16 rt][N2 + 4]
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int row = lane & 15, kk = lane >> 4;
  const int64_t x = blockIdx.x / groups;
  const int M1 = a.M[1], M2 = a.M[2], N1 = a.N[1], N2 = a.N[2], S = N2 + 4;
  const int r0 = (int)(blockIdx.x % groups) * rt, nr = min(rt, M1 / 16 - r0);
  for (int t = w; t < nr * (N2 / 16); t += kTrWaves) {
    const int r = t / (N2 / 16), c = t % (N2 / 16);
    const double* tp = a.tab[1] + 16 * (r0 + r);
    const double* ip = a.buf2 + x * N1 * N2 + 16 * c;
    const uint32_t to = 8 * (kk * M1 + row), io = 8 * (kk * N2 + row);
    v4d acc = {};
    tile_times(N1, [&](int k, int s) { return word_at(tp, 8u * (k + 4 * s) * M1 + to); },
               [&](int k, int s) { return word_at(ip, 8u * (k + 4 * s) * N2 + io); }, acc);
#pragma unroll
    for (int i = 0; i < 4; ++i) s_r[(16 * r + kk + 4 * i) * S + 16 * c + row] = acc[i];
  }
  __syncthreads();
  const int jt = (M2 + 63) / 64;
  for (int t = w; t < nr * jt; t += kTrWaves) {
    const int r = t / jt, j0 = t % jt * 64, nj = min(4, (M2 - j0) / 16);
    const double* ap = s_r + (16 * r + row) * S + 4 * kk;
    const double* tp = a.tab[2] + j0;
    const uint32_t to = 8 * (4 * kk * M2 + row);
    v4d acc[4] = {};
    rows_times<4, 2>(N2, [&](int k) { return *reinterpret_cast<const double4*>(ap + k); },
                  [&](int k, double (&v)[4][4]) {
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                      for (int c = 0; c < 4; ++c) v[s][c] = word_at(tp, 8u * ((k + s) * M2 + 16 * min(c, nj - 1)) + to);
                  }, acc);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (c >= nj) break;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        a.pot[(x * M1 + 16 * (r0 + r) + kk + 4 * i) * M2 + j0 + 16 * c + row] = acc[c][i];
    }
  }
}

// Sums of three values over a wave in a fixed order: x in lane 0, z in lanes 16 and 48, y in
// lane 32. The halves of the wave, then its rows, exchange what the other one keeps
// (v_permlane32_swap, v_permlane16_swap), so one sum over 16 lanes does for all three.
__device__ inline float wave_sum3(float x, float y, float z) {
  auto swap32 = [](float p, float q) {
    const auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(p), __float_as_uint(q), false, false);
    return __uint_as_float(v[0]) + __uint_as_float(v[1]);
  };
  const float xy = swap32(x, y), zz = swap32(z, z);
  const auto v = __builtin_amdgcn_permlane16_swap(__float_as_uint(xy), __float_as_uint(zz), false, false);
  float t = __uint_as_float(v[0]) + __uint_as_float(v[1]);
  auto dpp = [](float a, auto ctrl) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        0, __builtin_bit_cast(int, a), decltype(ctrl)::value, 0xf, 0xf, false));
  };
  t += dpp(t, std::integral_constant<int, 0xB1>());    // xor 1
  t += dpp(t, std::integral_constant<int, 0x4E>());    // xor 2
  t += dpp(t, std::integral_constant<int, 0x141>());   // mirror within 8
  t += dpp(t, std::integral_constant<int, 0x140>());   // mirror within 16
  return t;
}

// Forces, one workgroup of 8 (4 on the largest grids) waves per tile: the potential's coefficients around the tile
// (17 x 17 x 25 points) in LDS, in float32 less the value at the tile's corner; a wave takes an atom of the tile's bin at a time, its lanes the
// 100 (x, y) rows of the window (two rounds), each summing its row's 10 z values from both ends
// with phi_z and phi_z' (uniform, in scalar registers). The coefficient at the atom's own grid
// point is taken off every value: a constant exerts no force, and the derivative's rounding
// then scales with the potential's change over the window, not with the potential. Bound by
// instruction issue, about 200 per atom. 92,224 atoms: 54.6 us with 4 waves and a sum per
// component; 49.2 with one sum for the three; 46.9 with the buffer's old force read an atom
// ahead; 39.7 with 8 waves (more than four workgroups do not fit a compute unit's LDS, and
// four of 8 waves fill it; 10, 12 and 16 waves 47, 43 and 43); 41.3 with the potential read in float64.
template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_em_force(EwMeshArgs a) {
  constexpr int kRX = kTX + kW - 1, kRZ = kTZ + kW - 1;   // points around the tile
  constexpr int kQuads = (kRZ + 3) / 4;                   // 32-byte loads per row
  __shared__ float s_c[kRX * kRX * kRZ];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const int bin = blockIdx.x;
  const int tz = bin % a.nt[2], ty = (bin / a.nt[2]) % a.nt[1], tx = bin / (a.nt[2] * a.nt[1]);
  const int s0 = a.start[bin], s1 = a.start[bin + 1];
  if (s0 == s1) return;
  // rows start 4 points before a multiple of 16 on an axis of a multiple of 16, so a quad never
  // straddles the box edge and is aligned
  static_assert(kLo == 4 && kTZ % 4 == 0, "aligned quads");
  const double ref = a.pot[((int64_t)(kTX * tx) * a.M[1] + kTX * ty) * a.M[2] + kTZ * tz];
#pragma unroll 4
  for (int e = t; e < kRX * kRX * kQuads; e += kThreads) {
    const int qd = e % kQuads, rw = e / kQuads;
    int x = rw / kRX + kTX * tx - kLo, y = rw % kRX + kTX * ty - kLo, z = 4 * qd + kTZ * tz - kLo;
    x += x < 0 ? a.M[0] : x >= a.M[0] ? -a.M[0] : 0;
    y += y < 0 ? a.M[1] : y >= a.M[1] ? -a.M[1] : 0;
    z += z < 0 ? a.M[2] : z >= a.M[2] ? -a.M[2] : 0;
    const double4 v = *reinterpret_cast<const double4*>(&a.pot[((int64_t)x * a.M[1] + y) * a.M[2] + z]);
    float* d = s_c + rw * kRZ + 4 * qd;
    d[0] = (float)(v.x - ref);
    if (4 * qd + 1 < kRZ) {
      d[1] = (float)(v.y - ref);
      d[2] = (float)(v.z - ref);
      d[3] = (float)(v.w - ref);
    }
  }
  static_assert(kRZ % 4 == 1, "the last quad of a row holds one point");
  // this lane's window rows, and its part of an atom's windows: lane 10 d + k point k of axis d
  const bool in1 = lane + 64 < kW * kW;
  const int i0 = lane / kW, j0 = lane % kW, i1 = in1 ? (lane + 64) / kW : 0,
            j1 = in1 ? (lane + 64) % kW : 0;
  const int r0 = (i0 * kRX + j0) * kRZ, r1 = (i1 * kRX + j1) * kRZ;
  // wave_sum3 leaves the sums in lanes 0, 16 and 32
  const bool writes = (lane & 15) == 0 && lane < 48;
  const int axis = lane < 16 ? 0 : lane < 32 ? 2 : 1;
  const double mL = a.mL[axis];
  float* out = nullptr;
  float v = 0.f, held = 0.f;
  const int wl = min(lane, 31);
  uint4 u = make_uint4(0, 0, 0, 0);
  float wv = 0.f, dw = 0.f;
  int id = 0;
  auto fetch = [&](int s) {
    s = min(s, s1 - 1);
    u = a.rec[s];
    wv = a.win[(int64_t)s * 32 + wl];
    dw = a.dwin[(int64_t)s * 32 + wl];
    id = a.sid[s];
  };
  fetch(s0 + w);
  __syncthreads();
  for (int s = s0 + w; s < s1; s += kThreads / 64) {
    const int64_t at = 3 * (int64_t)id;
    uint32_t f;
    const int l = ((grid_cell(u.x, a.M[0], f) % kTX) * kRX + grid_cell(u.y, a.M[1], f) % kTX) * kRZ +
                  grid_cell(u.z, a.M[2], f) % kTZ;
    float wz[kW], dz[kW];
#pragma unroll
    for (int z = 0; z < kW; ++z) {
      wz[z] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wv), 2 * kW + z));
      dz[z] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(dw), 2 * kW + z));
    }
    const float wx0 = __shfl(wv, i0), dx0 = __shfl(dw, i0), wy0 = __shfl(wv, kW + j0),
                dy0 = __shfl(dw, kW + j0);
    const float wx1 = __shfl(wv, i1), dx1 = __shfl(dw, i1), wy1 = __shfl(wv, kW + j1),
                dy1 = __shfl(dw, kW + j1);
    fetch(s + kThreads / 64);
    const float cm = s_c[l + (kLo * kRX + kLo) * kRZ + kLo];
    const float *ca = s_c + l + r0, *cb = s_c + l + r1;
    float p0[2] = {0.f, 0.f}, z0[2] = {0.f, 0.f}, p1[2] = {0.f, 0.f}, z1[2] = {0.f, 0.f};
#pragma unroll
    for (int z = 0; z < kW / 2; ++z) {
      const int y = kW - 1 - z;
      const float va = ca[z] - cm, vb = ca[y] - cm, vc = cb[z] - cm, vd = cb[y] - cm;
      p0[0] = fmaf(va, wz[z], p0[0]);
      p0[1] = fmaf(vb, wz[y], p0[1]);
      z0[0] = fmaf(va, dz[z], z0[0]);
      z0[1] = fmaf(vb, dz[y], z0[1]);
      p1[0] = fmaf(vc, wz[z], p1[0]);
      p1[1] = fmaf(vd, wz[y], p1[1]);
      z1[0] = fmaf(vc, dz[z], z1[0]);
      z1[1] = fmaf(vd, dz[y], z1[1]);
    }
    const float pa = p0[0] + p0[1], pb = in1 ? p1[0] + p1[1] : 0.f;
    const float za = z0[0] + z0[1], zb = in1 ? z1[0] + z1[1] : 0.f;
    const float F = wave_sum3(fmaf(dx0 * wy0, pa, dx1 * wy1 * pb), fmaf(wx0 * dy0, pa, wx1 * dy1 * pb),
                              fmaf(wx0 * wy0, za, wx1 * wy1 * zb));
    if (writes) {
      // added to what the buffer holds an atom later, when the load is back
      if (out) *out = a.accumulate ? held + v : v;
      out = a.force + at + axis;
      v = (float)((double)F * mL);
      if (a.accumulate) held = *out;
    }
  }
  if (out) *out = a.accumulate ? held + v : v;
}

__global__ __launch_bounds__(256) void k_em_energy(EwMeshArgs a) {
  ew_energy_sum(a.epart, a.nepart, a.qpart, a.qblocks, a.L, a.alpha, a.coulomb_k, a.energy);
}

}  // namespace

static void mesh_sizes(const int32_t kmax[3], EwMeshPlan* pl) {
  for (int d = 0; d < 3; ++d) {
    const int K = kmax[d];
    pl->K[d] = K;
    pl->N[d] = (2 * (K + 1) + 15) / 16 * 16;
    int M = ((int)ceil(1.75 * (2 * K + 1)) + 15) / 16 * 16;
    const int least = d == 2 ? 3 * kTZ : 2 * kTZ;   // at least three tiles on every axis
    pl->M[d] = M < least ? least : M;
    pl->nt[d] = pl->M[d] / (d == 2 ? kTZ : kTX);
  }
  pl->nbins = (int64_t)pl->nt[0] * pl->nt[1] * pl->nt[2];
}

// Which systems take the grid: those of at least so many atoms, by a model of both forms' times in
// microseconds,
//   direct  26 + n x (rows and mz, up to multiples of 64) / 4e6
//   grid    42 + (operations of the transforms) / 3.5e7 + n x 0.57 / (tiles, at most 500)
// fitted to whole calls of 500 to 1,066,628 atoms with kmax 2 to 90 on each axis, and unequal ones up
// to 255. The direct sum's cost is in its products; the grid's in the transforms, whatever the
// atoms, and in the atoms of a tile, which one workgroup takes in turn: with few wave numbers there
// are 48 tiles, and no number of atoms makes it the faster one. Direct and grid, us:
//   kmax 4: 5,000 atoms 35 and 92, 92,224 130 and 1024, 1,066,628 724 and 12,603
//   kmax 12: 9,001 78 and 83, 92,224 447 and 494
//   kmax 16: 2,000 53 and 51, 9,001 108 and 63, 92,224 663 and 245
//   kmax 30: 1,000 72 and 82, 2,000 100 and 83, 40,000 1422 and 109
//   kmax 90: 500 489 and 1314, 3,000 2803 and 1371
// Of 160 points measured it picks the slower form at 2, by 5 and 17% (3,000 and 4,000 atoms). The tiles are taken
// as evenly filled: a system packed into a few of them takes the grid longer.
// Accuracy does not decide: the grid is the closer one to a float64 sum at all points compared, since the
// direct sum's float32 sums run over the atoms of a workgroup. RMS force error, direct and grid, alpha
// 0.3 at 0.1 atoms/A^3, with the wave numbers that alpha needs: 3,000 atoms 2.3e-7 and 8e-8, 40,000
// 1.05e-6 and 7.6e-8; with twice as many 9,001 8.2e-7 and 7.8e-8, with six times as many 2,500 1.7e-7
// and 8e-8; 33,880 in a 22 x 22 x 700 A box 5.3e-7 and 8.9e-8. Not under 2,000 atoms, nor where the grids take more than 512 MiB and more than the
// direct sum's phase tables.
int64_t ew_mesh_from(const int32_t kmax[3]) {
  EwMeshPlan pl;
  mesh_sizes(kmax, &pl);
  const double N[3] = {(double)pl.N[0], (double)pl.N[1], (double)pl.N[2]},
               M[3] = {(double)pl.M[0], (double)pl.M[1], (double)pl.M[2]};
  const double rows = kmax[0] * (2.0 * kmax[1] + 1) + kmax[1] + 1;
  const double direct = ceil(rows / 64) * 64 * ((2 * kmax[2] + 64) / 64) * 64 / 4e6;
  const double grid = 0.57 / (pl.nbins < 500 ? (double)pl.nbins : 500.0);
  if (direct <= grid) return INT64_MAX;
  const double ops = 4 * M[0] * (M[1] * M[2] * N[2] + M[1] * N[1] * N[2] + N[0] * N[1] * N[2]);
  double n = (16 + ops / 3.5e7) / (direct - grid);
  const double bytes = 8 * M[0] * (M[1] * M[2] + N[1] * N[2]);
  if (bytes > 536870912.0) n = fmax(n, bytes / (8.0 * (kmax[0] + 2 * kmax[1] + 2 * kmax[2] + 3)));
  return n < 2000 ? 2000 : (int64_t)ceil(n);
}

void ew_mesh_plan(int64_t n, const int32_t kmax[3], EwMeshPlan* pl) {
  mesh_sizes(kmax, pl);
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t nn = (size_t)n;
  const size_t M0 = pl->M[0], M1 = pl->M[1], M2 = pl->M[2], N0 = pl->N[0], N1 = pl->N[1], N2 = pl->N[2];
  size_t o = al(sizeof(WsHeader));
  // the fractions, bins and indices in the callers' order are done with when k_em_middle writes buf2
  pl->off_buf2 = pl->off_ups = o;
  pl->off_slot = pl->off_ups + al(16 * nn);
  pl->off_ids = pl->off_slot + al(8 * nn);
  const size_t atoms = al(16 * nn) + al(8 * nn) + al(4 * nn), back = al(8 * M0 * N1 * N2);
  o += atoms > back ? atoms : back;
  pl->off_rec = o;   o = al(o + 16 * nn);
  pl->off_win = o;   o = al(o + 128 * nn);
  pl->off_dwin = o;  o = al(o + 128 * nn);
  pl->off_sid = o;   o = al(o + 4 * nn);
  pl->off_count = o; o = al(o + 4 * (size_t)(mesh_pad(pl->nbins) * pl->nbins));
  pl->off_start = o; o = al(o + 4 * (size_t)(pl->nbins + 1));
  // the charges, and their transform along z and y (each axis has fewer modes than points), are done with
  // when k_em_back writes the potential
  pl->off_pot = pl->off_buf0 = o;
  pl->off_buf1 = o + 4 * M0 * M1 * M2;
  o = al(o + 8 * M0 * M1 * M2);
  for (int d = 0; d < 3; ++d) {
    const size_t e = (size_t)pl->N[d] * pl->M[d];
    pl->off_tab[d] = o;  o = al(o + 8 * e);
    pl->off_tabT[d] = o; o = al(o + 8 * e);
    pl->off_gfac[d] = o; o = al(o + 8 * (size_t)pl->N[d]);
    pl->off_ksq[d] = o;  o = al(o + 8 * (size_t)pl->N[d]);
  }
  pl->nepart = (int64_t)((N0 / 16) * (N1 * N2 / 16));
  pl->off_epart = o; o = al(o + 8 * (size_t)pl->nepart);
  pl->qblocks = (n + 255) / 256;
  pl->off_qpart = o; o = al(o + 16 * (size_t)pl->qblocks);
  pl->total = o;
}

hipError_t launch_ew_mesh(const EwMeshPlan& pl, const md_params* p, int64_t n, const float* pos,
                          const float* q, float* force, double* energy, int accumulate, void* ws,
                          hipStream_t st) {
  EwMeshArgs a;
  char* b = (char*)ws;
  a.n = n;
  a.pos = pos;
  a.q = q;
  a.force = force;
  a.energy = energy;
  a.accumulate = accumulate;
  a.hdr = (WsHeader*)b;
  a.ups = (uint4*)(b + pl.off_ups);
  a.rec = (uint4*)(b + pl.off_rec);
  a.win = (float*)(b + pl.off_win);
  a.dwin = (float*)(b + pl.off_dwin);
  a.slot = (int2*)(b + pl.off_slot);
  a.ids = (int*)(b + pl.off_ids);
  a.sid = (int*)(b + pl.off_sid);
  a.count = (int*)(b + pl.off_count);
  a.start = (int*)(b + pl.off_start);
  a.buf0 = (float*)(b + pl.off_buf0);
  a.pot = (double*)(b + pl.off_pot);
  a.buf1 = (float*)(b + pl.off_buf1);
  a.buf2 = (double*)(b + pl.off_buf2);
  a.epart = (double*)(b + pl.off_epart);
  a.qpart = (double2*)(b + pl.off_qpart);
  a.nepart = pl.nepart;
  a.qblocks = pl.qblocks;
  a.nbins = pl.nbins;
  a.pad = (int)mesh_pad(pl.nbins);
  a.alpha = p->ewald_alpha;
  a.coulomb_k = p->coulomb_k;
  double V = 1;
  int64_t entries = 0, modes = 0;
  for (int d = 0; d < 3; ++d) {
    a.M[d] = pl.M[d];
    a.N[d] = pl.N[d];
    a.K[d] = pl.K[d];
    a.nt[d] = pl.nt[d];
    a.L[d] = (double)(float)p->box[d];   // the float32 box
    a.mL[d] = (double)pl.M[d] / a.L[d];
    V *= a.L[d];
    a.tab[d] = (double*)(b + pl.off_tab[d]);
    a.tabT[d] = (double*)(b + pl.off_tabT[d]);
    a.gfac[d] = (double*)(b + pl.off_gfac[d]);
    a.ksq[d] = (double*)(b + pl.off_ksq[d]);
    entries += (int64_t)pl.N[d] * pl.M[d];
    modes += pl.N[d] / 2;
    // the window's shape for the axis's oversampling (no narrower past 2.5)
    const double sigma = fmin(2.5, (double)pl.M[d] / (2.0 * pl.K[d] + 1.0));
    a.cb[d] = kW * M_PI * (1.0 - 0.5 / sigma) * M_LOG2E;
  }
  a.gscale = 4.0 * M_PI * p->coulomb_k / V;
  const unsigned nb = (unsigned)((n + 255) / 256);
  const unsigned nb_tab = (unsigned)((entries + 255) / 256);
  hipLaunchKernelGGL(k_em_init, dim3(nb_tab + (unsigned)((modes + 3) / 4)), dim3(256), 0, st, a, nb_tab);
  hipLaunchKernelGGL(k_em_setup, dim3(nb), dim3(256), 0, st, a);
  if (a.nbins <= kPlaceBins) {
    hipLaunchKernelGGL(k_em_place, dim3((unsigned)((n + kPlaceThreads - 1) / kPlaceThreads)), dim3(kPlaceThreads),
                       0, st, a);
  } else {
    hipLaunchKernelGGL(k_em_scan, dim3(1), dim3(1024), 0, st, a);
    hipLaunchKernelGGL(k_em_scatter, dim3(nb), dim3(256), 0, st, a);
  }
  hipLaunchKernelGGL(k_em_sort, dim3((unsigned)pl.nbins), dim3(256), 0, st, a);
  hipLaunchKernelGGL(k_em_spread, dim3((unsigned)pl.nbins), dim3(256), 0, st, a);
  // workgroups of the transforms: four per compute unit where the tiles allow it (with one, 288
  // workgroups, 45 us for all three; with four 43, float32 products), at most two column tiles or
  // three row tiles each (with three column tiles 21 registers of k_em_forward spill: kmax (150, 40,
  // 40) 492 us for the whole sum, 471 with two) and 64 KB of LDS (a kmax of 255 makes an axis of 896
  // points and 512 modes)
  const int need = (1024 + a.M[0] - 1) / a.M[0];
  auto share = [&](int tiles, int most, auto bytes, int& groups) {
    int c = (tiles + need - 1) / need;
    c = c > most ? most : c;
    while (c > 1 && bytes(c) > 65536) --c;
    groups = (tiles + c - 1) / c;
    return (tiles + groups - 1) / groups;
  };
  int gf, gb;
  auto fb = [&](int c) { return (size_t)64 * a.M[1] * (c | 1); };
  auto bb = [&](int c) { return (size_t)128 * c * (a.N[2] + 4); };
  const int cf = share(a.N[2] / 16, 2, fb, gf), rt = share(a.M[1] / 16, 3, bb, gb);
  const dim3 grid((unsigned)(a.M[0] * gf)), wg(kTrThreads);
  if (cf == 1) hipLaunchKernelGGL(k_em_forward<1>, grid, wg, fb(1), st, a, gf);
  else hipLaunchKernelGGL(k_em_forward<2>, grid, wg, fb(2), st, a, gf);
  hipLaunchKernelGGL(k_em_middle, dim3((unsigned)(a.N[1] * a.N[2] / 16)), wg, (size_t)64 * a.N[0], st, a);
  hipLaunchKernelGGL(k_em_back, dim3((unsigned)(a.M[0] * gb)), wg, bb(rt), st, a, rt, gb);
  // 8 waves a tile, but 4 on the largest grids, whose tiles hold a few atoms each while their
  // staging reads past the caches: five workgroups of 4 waves fit a compute unit, four of 8.
  // Whole sums with 8 and with 4: 92,224 atoms in 2,268 bins 149 and 156 us, 40,000 in 16,384 467
  // and 479, 100,000 in 32,000 1128 and 1078, 30,000 in 32,000 959 and 962.
  if (a.nbins > 24576) hipLaunchKernelGGL(k_em_force<256>, dim3((unsigned)pl.nbins), dim3(256), 0, st, a);
  else hipLaunchKernelGGL(k_em_force<512>, dim3((unsigned)pl.nbins), dim3(512), 0, st, a);
  hipLaunchKernelGGL(k_em_energy, dim3(1), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace md
