// Ewald reciprocal-space sum: the Coulomb energy and forces beyond the short-range kernel.
//
// Section 2.1 splits the non-bonded work at the cutoff and hands the Coulomb part beyond
// it to an approximation outside the short-range kernel. Read here as Ewald summation of
// the periodic box: the short-range kernel (MD_COULOMB_EWALD) evaluates the screened term
// k q_i q_j erfc(alpha r)/r inside the cutoff, and this file the smooth rest,
//   E_recip = (4 pi k / V) sum_{half space of kv} w(kv) |S(kv)|^2,
//   w(kv)   = exp(-|kv|^2 / (4 alpha^2)) / |kv|^2,   S(kv) = sum_j q_j exp(i kv . r_j),
//   F_i     = q_i sum_{half space} kv Im(G(kv) exp(i kv . r_i)),  G = (8 pi k / V) w conj(S),
// over kv = 2 pi (mx/Lx, my/Ly, mz/Lz) with |m_d| <= kmax_d, one of each pair +-kv (the
// two give equal terms), plus the self term -k alpha/sqrt(pi) sum q^2 and the neutralising
// background -k pi Q^2 / (2 V alpha^2).
//
// This file holds the entry points and the direct sum, which systems of few atoms or few wave
// numbers take; the others take the same sum through a grid (md_ewald_mesh.hip, ew_mesh_from).
//
// Phases are exact modulo one turn: each atom's fractional coordinate is held as a 32-bit
// fixed-point fraction u, so m u (mod 2^32) is the phase of wave number m with no rounding,
// and only the final sine and cosine round. Wave vectors are grouped in rows (mx, my), each
// row holding every mz; the kernels are
//   k_ew_prepare  per atom: fractions u, charge, NaN check, partial sums of q^2 and q; and per
//                 atom and wave number exp(2 pi i m u) per axis, float2 [m][atom];
//   k_ew_sf       structure factors as a complex matrix product over atoms on the matrix cores
//                 (W = q X Y per (row, atom), Z per (atom, mz)); per-chunk partial sums;
//   k_ew_g        G from the chunks' partials (float64, eight loads in flight), row energies;
//   k_ew_force    per 64 atoms and a share of the rows: T = Z G over mz on the matrix cores and
//                 one sine/cosine of the exact (mx, my) phase per atom and row;
//   k_ew_final    the shares of an atom's force added; fixed-order sum of the row energies, self
//                 and background, and the status word.
// Most systems that come here are small (larger ones with many wave numbers take the grid), so
// launches and idle compute units count: 3,000 atoms and 6,095 wave vectors took seven launches, 47 workgroups for the
// forces and 47 dependent loads per wave vector, 89 us; 41 this way, the same bits.
// Every sum runs in a fixed order, so the results are the same bits on every run.
#include <math.h>

#include "md_ewald.hpp"

namespace md {
namespace {

constexpr int kEwTile = 64;       // atoms per LDS tile of the structure-factor kernel
constexpr int kEwRows = 64;       // rows per structure-factor workgroup (4 tiles of 16)
constexpr int kEwZ = 64;          // mz values per chunk of the force kernel (A operands in
                                  // registers), and the padding of G's rows
constexpr int kEwMaxK = 255;      // largest kmax per axis

struct EwArgs {
  int64_t n;
  const float* pos;               // [n][3], caller order
  const float* q;                 // [n]
  float* force;                   // [n][3]
  double* energy;                 // [1]
  int accumulate;
  WsHeader* hdr;
  uint4* ups;                     // [n]: fractions ux, uy, uz and the charge's bits
  float2* tab;                    // [(kx+1) + (2ky+1) + (2kz+1)][n]: X, then Y, then Z
  float2* parts;                  // [chunks][R][nzc] partial structure factors
  float2* g;                      // [R][nzc_pad] G (zero where excluded and in the padding)
  double* fpart;                  // [splits][n][3] shares of the forces (splits > 1), where parts was
  uint32_t* stat;                 // [qblocks] status bits
  double* erow;                   // [R][zblocks] energy partials
  double2* qpart;                 // [qblocks] (sum q^2, sum q) per setup block
  int kx, ky, kz, nzc, nzc_pad, zblocks;
  int splits, split_rows;         // shares of the rows in k_ew_force, rows (of 16) in each
  int64_t rows, chunks, chunk_atoms, qblocks;
  double L[3];
  double alpha, coulomb_k;
};

__host__ __device__ inline int64_t ew_rows(int kx, int ky) {
  return (int64_t)kx * (2 * ky + 1) + (ky + 1);
}

// Row r -> (mx, my): rows 0..ky are (0, my >= 0), then mx >= 1 with every my.
__device__ inline void ew_row(const EwArgs& a, int64_t r, int& mx, int& my) {
  if (r <= a.ky) {
    mx = 0;
    my = (int)r;
  } else {
    const int64_t s = r - (a.ky + 1);
    mx = 1 + (int)(s / (2 * a.ky + 1));
    my = (int)(s % (2 * a.ky + 1)) - a.ky;
  }
}

// exp(2 pi i m u / 2^32) for the phase m u taken modulo 2^32 (exact), as (cos, sin).
__device__ inline float2 ew_phase(uint32_t ph) {
  float s, c;
  sincospif((float)(int32_t)ph * 4.656612873077393e-10f, &s, &c);   // 2^-31: units of pi
  return make_float2(c, s);
}

// Table row t = blockIdx.y: X (mx = 0..kx), Y (my = -ky..ky), Z (mz = -kz..kz), each [m][atom];
// the blocks of row 0 also write the atoms' fractions and partial sums.
__global__ __launch_bounds__(256) void k_ew_prepare(EwArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int t = blockIdx.y;
  if (i < a.n) {
    int m, d;
    if (t <= a.kx) {
      m = t;
      d = 0;
    } else if (t <= a.kx + 2 * a.ky + 1) {
      m = t - (a.kx + 1) - a.ky;
      d = 1;
    } else {
      m = t - (a.kx + 2 * a.ky + 2) - a.kz;
      d = 2;
    }
    uint32_t st = 0;
    a.tab[(int64_t)t * a.n + i] = ew_phase((uint32_t)m * ew_fraction(a.pos[3 * i + d], a.L[d], st));
  }
  if (t > 0) return;
  double q2 = 0.0, q1 = 0.0;
  uint32_t st = 0;
  if (i < a.n) {
    const uint4 u = ew_fractions(a.pos, a.q, a.L, i, st);
    a.ups[i] = u;
    const double qi = (double)__uint_as_float(u.w);
    q2 = qi * qi;
    q1 = qi;
  }
  __shared__ double s_q2[4], s_q1[4];
  __shared__ uint32_t s_st[4];
  for (int off = 32; off > 0; off >>= 1) {
    q2 += __shfl_xor(q2, off);
    q1 += __shfl_xor(q1, off);
    st |= __shfl_xor(st, off);
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    s_q2[w] = q2;
    s_q1[w] = q1;
    s_st[w] = st;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    a.qpart[blockIdx.x] = make_double2((s_q2[0] + s_q2[1]) + (s_q2[2] + s_q2[3]),
                                       (s_q1[0] + s_q1[1]) + (s_q1[2] + s_q1[3]));
    a.stat[blockIdx.x] = s_st[0] | s_st[1] | s_st[2] | s_st[3];
  }
}

// Structure factors as a complex matrix product over atoms, on the matrix cores:
// S[r][mz] = sum_j W[r][j] Z[j][mz], W = q X[mx(r)] Y[my(r)]. A workgroup takes 64 rows x
// 64 values of mz x one chunk of atoms; wave w owns the 16 x 16 output tile (rows
// 16 (w / 4) .., mz 16 (w % 4) ..). Per tile of 64 atoms the workgroup writes W (computed)
// and Z (loaded) to LDS, atom-major and padded so that both the transposing stores and the
// operand reads spread over the banks; each wave then runs 16 steps of 4 atoms, each step
// four v_mfma_f32_16x16x4f32 (re re, -im im, re im, im re). In a 16x16x4 f32 product, lane
// l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and holds D[4 (l / 16) + i][l % 16],
// i = 0..3. The accumulation order is fixed, so the partial sums are the same bits on every
// run.
typedef float ew_v4f __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_ew_sf(EwArgs a) {
  __shared__ float2 sW[kEwTile][kEwRows + 1];   // [atom][row]
  __shared__ float2 sZ[kEwTile][64 + 1];        // [atom][mz]
  const int t = threadIdx.x;
  const int w = t >> 6, lane = t & 63;
  const int64_t r0 = (int64_t)blockIdx.x * kEwRows;
  const int z0 = blockIdx.z * 64;
  const int64_t a0 = (int64_t)blockIdx.y * a.chunk_atoms;
  const int64_t a1 = a0 + a.chunk_atoms < a.n ? a0 + a.chunk_atoms : a.n;
  // staging roles: atom ta = t % 64 of the tile; W for rows 4 (t / 64) .. + 3, Z for mz
  // t / 64 + 16 p (p = 0..3)
  const int ta = t & 63, tg = t >> 6;
  int mxs[4], mys[4];
  bool rok[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t r = r0 + 4 * tg + k;
    rok[k] = r < a.rows;
    mxs[k] = 0;
    mys[k] = 0;
    if (rok[k]) ew_row(a, r, mxs[k], mys[k]);
  }
  const float2* Z = a.tab + (int64_t)(a.kx + 2 * a.ky + 2) * a.n;
  // this wave's output tile and its operand columns
  const int rt = w >> 2, zt = w & 3;
  const int ar = 16 * rt + (lane & 15);   // A row (this lane's row of W)
  const int bz = 16 * zt + (lane & 15);   // B column (this lane's mz)
  const int kk = lane >> 4;               // this lane's atom within a step
  ew_v4f dre = {0.f, 0.f, 0.f, 0.f}, dim = {0.f, 0.f, 0.f, 0.f};
  // this thread's staging values of one tile, loaded a tile ahead of their use
  float2 wn[4], zn[4];
  auto load_tile = [&](int64_t t0) __attribute__((always_inline)) {
    const int64_t j = t0 + ta;
    const bool jok = j < a1;
    const float qj = jok ? __uint_as_float(a.ups[j].w) : 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float2 wv = make_float2(0.f, 0.f);
      if (jok && rok[k]) {
        const float2 x = a.tab[(int64_t)mxs[k] * a.n + j];
        const float2 y = a.tab[(int64_t)(a.kx + 1 + mys[k] + a.ky) * a.n + j];
        wv = make_float2(qj * (x.x * y.x - x.y * y.y), qj * (x.x * y.y + x.y * y.x));
      }
      wn[k] = wv;
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int zi = z0 + tg + 16 * p;
      zn[p] = (jok && zi < a.nzc) ? Z[(int64_t)zi * a.n + j] : make_float2(0.f, 0.f);
    }
  };
  if (a0 < a1) load_tile(a0);
  for (int64_t t0 = a0; t0 < a1; t0 += kEwTile) {
#pragma unroll
    for (int k = 0; k < 4; ++k) sW[ta][4 * tg + k] = wn[k];
#pragma unroll
    for (int p = 0; p < 4; ++p) sZ[ta][tg + 16 * p] = zn[p];
    __syncthreads();
    if (t0 + kEwTile < a1) load_tile(t0 + kEwTile);
    // atoms past the chunk's end hold W = Z = 0, so every step can run in full
#pragma unroll 4
    for (int s = 0; s < kEwTile / 4; ++s) {
      const float2 av = sW[4 * s + kk][ar];
      const float2 bv = sZ[4 * s + kk][bz];
      dre = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, bv.x, dre, 0, 0, 0);
      dre = __builtin_amdgcn_mfma_f32_16x16x4f32(-av.y, bv.y, dre, 0, 0, 0);
      dim = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, bv.y, dim, 0, 0, 0);
      dim = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, bv.x, dim, 0, 0, 0);
    }
    __syncthreads();
  }
  const int zi = z0 + bz;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t r = r0 + 16 * rt + 4 * kk + i;
    if (r < a.rows && zi < a.nzc)
      a.parts[((int64_t)blockIdx.y * a.rows + r) * a.nzc + zi] = make_float2(dre[i], dim[i]);
  }
}

// G of wave vector (row r, mz index zi) from the chunks' partials (fixed order, float64), zero
// outside the half space kv != 0; e gets its energy term.
__device__ inline float2 ew_g(const EwArgs& a, int64_t r, int zi, double& e) {
  e = 0.0;
  if (r >= a.rows || zi >= a.nzc) return make_float2(0.f, 0.f);
  int mx, my;
  ew_row(a, r, mx, my);
  const int mz = zi - a.kz;
  if (!(mx > 0 || my > 0 || mz > 0)) return make_float2(0.f, 0.f);
  double sr = 0.0, si = 0.0;
  const float2* p = a.parts + r * a.nzc + zi;
  const int64_t step = a.rows * a.nzc;
  for (int64_t c = 0; c < a.chunks; c += 8) {
    float2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[(c + u < a.chunks ? c + u : a.chunks - 1) * step];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (c + u < a.chunks) {
        sr += (double)v[u].x;
        si += (double)v[u].y;
      }
    }
  }
  const double pi = 3.141592653589793;
  const double kx = 2.0 * pi * mx / a.L[0], ky = 2.0 * pi * my / a.L[1],
               kz = 2.0 * pi * mz / a.L[2];
  const double k2 = kx * kx + ky * ky + kz * kz;
  const double wk = exp(-k2 / (4.0 * a.alpha * a.alpha)) / k2;
  const double V = a.L[0] * a.L[1] * a.L[2];
  e = 4.0 * pi * a.coulomb_k / V * wk * (sr * sr + si * si);
  const double gs = 8.0 * pi * a.coulomb_k / V * wk;
  return make_float2((float)(gs * sr), (float)(-gs * si));   // (8 pi k / V) w conj(S)
}

// G, and the rows' energies: a wave per row and 64 values of mz.
__global__ __launch_bounds__(256) void k_ew_g(EwArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= a.rows) return;
  const int zi = blockIdx.y * 64 + lane;
  double e;
  const float2 g = ew_g(a, r, zi, e);
  if (zi < a.nzc_pad) a.g[r * a.nzc_pad + zi] = g;
  for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off);
  if (lane == 0) a.erow[r * a.zblocks + blockIdx.y] = e;
}

// Atom i's force, from float64 sums without its charge.
__device__ inline void ew_put_force(const EwArgs& a, int64_t i, const double (&F)[3]) {
  const double qi = (double)__uint_as_float(a.ups[i].w);
  float* out = a.force + 3 * i;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float v = (float)(qi * F[d]);
    out[d] = a.accumulate ? out[d] + v : v;
  }
}

// Forces as complex matrix products over mz, on the matrix cores: for atoms i and rows
// (mx, my), T[i][r] = sum_mz Z[mz][i] G[r][mz] and U[i][r] = sum_mz mz Z[mz][i] G[r][mz];
// then F_i = q_i sum_r (kx, ky) Im(xy T) + (0, 0, kz) Im(xy U) with xy = exp(i (kx x + ky
// y)) from the exact phase of (mx, my). A workgroup of 4 waves takes 64 atoms, a wave 16 of
// them (rows of A, Z of its atoms for 64 values of mz in registers) against tiles of 16
// rows of G (columns of B) staged in LDS; each step of 4 values of mz runs eight
// v_mfma_f32_16x16x4f32 (T and U, re and im parts). A lane then holds 4 atoms x 1 row of T
// and U: it adds that row's force terms for its 4 atoms in float32 and each tile's sums into
// float64; the 16 lanes of a row group finally add their sums in a fixed butterfly.
// Three waves per SIMD (at most 168 registers): 40,000 atoms and kmax 27 806 us at two, 655 at three.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_ew_force(EwArgs a) {
  __shared__ float2 sG[16][kEwZ + 1];   // [row][mz] of the current tile and mz chunk
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const int kk = lane >> 4, col = lane & 15;
  const int64_t ia = (int64_t)blockIdx.x * 64 + 16 * w + col;   // this lane's A row (atom)
  const bool aok = ia < a.n;
  // the 4 atoms of this lane's D rows: 16 w + 4 kk + i
  uint32_t ux[4], uy[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t id = (int64_t)blockIdx.x * 64 + 16 * w + 4 * kk + i;
    const uint4 u = id < a.n ? a.ups[id] : make_uint4(0, 0, 0, 0);
    ux[i] = u.x;
    uy[i] = u.y;
  }
  const double pi = 3.141592653589793;
  const float kxs = (float)(2.0 * pi / a.L[0]), kys = (float)(2.0 * pi / a.L[1]),
              kzs = (float)(2.0 * pi / a.L[2]);
  double F[4][3] = {};
  const int64_t row0 = (int64_t)blockIdx.y * a.split_rows,
                row1 = row0 + a.split_rows < a.rows ? row0 + a.split_rows : a.rows;
  const float2* Zt = a.tab + (int64_t)(a.kx + 2 * a.ky + 2) * a.n;
  for (int zc = 0; zc < a.nzc_pad; zc += kEwZ) {
    // A operands for this mz chunk: step s holds Z[zc + 4 s + kk][ia]; ns steps cover the
    // chunk's mz values below nzc
    const int ns = (min(kEwZ, a.nzc - zc) + 3) / 4;
    float2 z[kEwZ / 4];
#pragma unroll
    for (int s = 0; s < kEwZ / 4; ++s) {
      const int zi = zc + 4 * s + kk;
      z[s] = (aok && zi < a.nzc) ? Zt[(int64_t)zi * a.n + ia] : make_float2(0.f, 0.f);
    }
    for (int64_t r0 = row0; r0 < row1; r0 += 16) {
      __syncthreads();
#pragma unroll
      for (int rr = w; rr < 16; rr += 4)   // a wave per row
        sG[rr][lane] = r0 + rr < a.rows ? a.g[(r0 + rr) * a.nzc_pad + zc + lane] : make_float2(0.f, 0.f);
      __syncthreads();
      ew_v4f tre = {0.f, 0.f, 0.f, 0.f}, tim = tre, ure = tre, uim = tre;
#pragma unroll
      for (int s = 0; s < kEwZ / 4; ++s) {
        if (s < ns) {   // steps past the chunk's last mz are skipped (uniform)
          const float2 g = sG[col][4 * s + kk];
          const float mz = (float)(zc + 4 * s + kk - a.kz);
          const float2 gm = make_float2(mz * g.x, mz * g.y);
          tre = __builtin_amdgcn_mfma_f32_16x16x4f32(z[s].x, g.x, tre, 0, 0, 0);
          tre = __builtin_amdgcn_mfma_f32_16x16x4f32(-z[s].y, g.y, tre, 0, 0, 0);
          tim = __builtin_amdgcn_mfma_f32_16x16x4f32(z[s].x, g.y, tim, 0, 0, 0);
          tim = __builtin_amdgcn_mfma_f32_16x16x4f32(z[s].y, g.x, tim, 0, 0, 0);
          ure = __builtin_amdgcn_mfma_f32_16x16x4f32(z[s].x, gm.x, ure, 0, 0, 0);
          ure = __builtin_amdgcn_mfma_f32_16x16x4f32(-z[s].y, gm.y, ure, 0, 0, 0);
          uim = __builtin_amdgcn_mfma_f32_16x16x4f32(z[s].x, gm.y, uim, 0, 0, 0);
          uim = __builtin_amdgcn_mfma_f32_16x16x4f32(z[s].y, gm.x, uim, 0, 0, 0);
        }
      }
      // this lane's row r0 + col against its 4 atoms (rows past the end hold T = U = 0)
      const int64_t r = r0 + col;
      int mx = 0, my = 0;
      if (r < a.rows) ew_row(a, r, mx, my);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 xy = ew_phase((uint32_t)mx * ux[i] + (uint32_t)my * uy[i]);
        const float imt = fmaf(xy.x, tim[i], xy.y * tre[i]);   // Im(xy T)
        const float imu = fmaf(xy.x, uim[i], xy.y * ure[i]);   // Im(xy U)
        F[i][0] += (double)((float)mx * kxs * imt);
        F[i][1] += (double)((float)my * kys * imt);
        F[i][2] += (double)(kzs * imu);
      }
    }
  }
  // sum over the 16 lanes of each row group (fixed butterfly), then lane 16 kk + 0 writes
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int sft = 1; sft < 16; sft <<= 1) F[i][d] += __shfl_xor(F[i][d], sft);
  if (col == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t id = (int64_t)blockIdx.x * 64 + 16 * w + 4 * kk + i;
      if (id >= a.n) continue;
      if (a.splits > 1) {
        double* out = a.fpart + 3 * ((int64_t)blockIdx.y * a.n + id);
        for (int d = 0; d < 3; ++d) out[d] = F[i][d];
      } else {
        ew_put_force(a, id, F[i]);
      }
    }
  }
}

// Block 0: the energy (row partials, then self and background terms) and the status word;
// blocks 1 ..: the shares of each atom's force added in a fixed order.
__global__ __launch_bounds__(256) void k_ew_final(EwArgs a) {
  if (blockIdx.x == 0) {
    __shared__ uint32_t s_st;
    if (threadIdx.x == 0) s_st = 0;
    __syncthreads();
    uint32_t st = 0;
    for (int64_t b = threadIdx.x; b < a.qblocks; b += 256) st |= a.stat[b];
    if (st) atomicOr(&s_st, st);
    ew_energy_sum(a.erow, a.rows * a.zblocks, a.qpart, a.qblocks, a.L, a.alpha, a.coulomb_k, a.energy);
    if (threadIdx.x == 0) a.hdr->status = s_st;   // past the sum's barriers
    return;
  }
  const int64_t i = ((int64_t)blockIdx.x - 1) * 256 + threadIdx.x;
  if (i >= a.n) return;
  double F[3] = {};
  for (int c = 0; c < a.splits; ++c)
#pragma unroll
    for (int d = 0; d < 3; ++d) F[d] += a.fpart[3 * ((int64_t)c * a.n + i) + d];
  ew_put_force(a, i, F);
}

struct EwPlan {
  int kx, ky, kz, nzc, nzc_pad, zblocks;
  int splits, split_rows;
  int64_t rows, chunks, chunk_atoms, qblocks;
  size_t off_ups, off_tab, off_parts, off_g, off_erow, off_qpart, off_stat, total;
};

size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

md_status ew_plan(const md_params* p, int64_t n, const int32_t kmax[3], EwPlan* pl) {
  if (!p || !kmax || n < 0 || n > kMaxAtoms) return MD_ERR_INVALID_ARG;
  if (!(p->ewald_alpha > 0) || !isfinite(p->ewald_alpha) || !isfinite(p->coulomb_k))
    return MD_ERR_INVALID_ARG;
  for (int d = 0; d < 3; ++d) {
    if (!(p->box[d] > 0) || !isfinite(p->box[d])) return MD_ERR_INVALID_ARG;
    if (kmax[d] < 0 || kmax[d] > kEwMaxK) return MD_ERR_INVALID_ARG;
  }
  if (kmax[0] + kmax[1] + kmax[2] == 0) return MD_ERR_INVALID_ARG;
  pl->kx = kmax[0];
  pl->ky = kmax[1];
  pl->kz = kmax[2];
  pl->nzc = 2 * pl->kz + 1;
  pl->nzc_pad = (pl->nzc + kEwZ - 1) / kEwZ * kEwZ;
  pl->zblocks = (pl->nzc_pad + 63) / 64;
  pl->rows = ew_rows(pl->kx, pl->ky);
  // atom chunks: enough workgroups to fill the chip, chunks of whole tiles
  const int64_t rb = (pl->rows + kEwRows - 1) / kEwRows;
  const int64_t tiles = (n + kEwTile - 1) / kEwTile > 0 ? (n + kEwTile - 1) / kEwTile : 1;
  int64_t chunks = (512 + rb * pl->zblocks - 1) / (rb * pl->zblocks);   // two per compute unit
  chunks = chunks < 1 ? 1 : chunks > tiles ? tiles : chunks;
  const int64_t most_chunks = chunks;
  pl->chunk_atoms = (tiles + chunks - 1) / chunks * kEwTile;
  pl->chunks = n > 0 ? (n + pl->chunk_atoms - 1) / pl->chunk_atoms : 1;
  pl->qblocks = (n + 255) / 256 > 0 ? (n + 255) / 256 : 1;
  // shares of the rows in the force kernel: about two workgroups per compute unit
  const int64_t at = (n + 63) / 64 > 0 ? (n + 63) / 64 : 1, rt = (pl->rows + 15) / 16;
  int64_t splits = (512 + at - 1) / at;
  splits = splits > rt ? rt : splits;
  pl->split_rows = (int)((rt + splits - 1) / splits * 16);
  pl->splits = (int)((pl->rows + pl->split_rows - 1) / pl->split_rows);
  const size_t nn = (size_t)(n > 0 ? n : 1);
  const int64_t trows = (pl->kx + 1) + (2 * pl->ky + 1) + pl->nzc;
  size_t o = a256(sizeof(WsHeader));
  pl->off_ups = o;   o = a256(o + sizeof(uint4) * nn);
  pl->off_tab = o;   o = a256(o + sizeof(float2) * (size_t)trows * nn);
  // the partial structure factors, and after them the shares of the forces in the same place. Both by
  // bounds that never fall as n grows (the chunks before they are evened out; splits x n, with splits at most
  // 512 / at + 1 and one share only from 32,768 atoms on), so that a workspace holds every smaller system
  const int64_t shares = rt == 1 ? 0 : rt * at < 512 + at ? rt * at : at < 512 ? 512 + at : 1024;   // of 64 atoms
  const size_t part_bytes = sizeof(float2) * (size_t)most_chunks * pl->rows * pl->nzc;
  const size_t share_bytes = sizeof(double) * 3 * 64 * (size_t)shares;
  pl->off_parts = o; o = a256(o + (part_bytes > share_bytes ? part_bytes : share_bytes));
  pl->off_g = o;     o = a256(o + sizeof(float2) * (size_t)pl->rows * pl->nzc_pad);
  pl->off_erow = o;  o = a256(o + sizeof(double) * (size_t)pl->rows * pl->zblocks);
  pl->off_qpart = o; o = a256(o + sizeof(double2) * (size_t)pl->qblocks);
  pl->off_stat = o;  o = a256(o + sizeof(uint32_t) * (size_t)pl->qblocks);
  pl->total = o;
  return MD_OK;
}

// Workspace of a call: it holds every call of fewer atoms too, whichever form those take.
size_t ew_bytes(const md_params* p, int64_t n, const int32_t kmax[3], const EwPlan* direct) {
  const int64_t from = ew_mesh_from(kmax);
  if (n < from) return direct->total;
  EwMeshPlan mesh;
  ew_mesh_plan(n, kmax, &mesh);
  EwPlan last;
  ew_plan(p, from - 1, kmax, &last);
  return mesh.total > last.total ? mesh.total : last.total;
}

}  // namespace
}  // namespace md

extern "C" {

size_t md_ewald_workspace_bytes(const md_params* p, int64_t n_atoms, const int32_t kmax[3]) {
  md::EwPlan pl;
  if (md::ew_plan(p, n_atoms, kmax, &pl) != MD_OK) return 0;
  return md::ew_bytes(p, n_atoms, kmax, &pl);
}

md_status md_ewald_recip_f32(const md_params* p, int64_t n_atoms, const float* d_pos,
                             const float* d_charge, const int32_t kmax[3], float* d_force,
                             double* d_energy, int32_t accumulate, void* d_ws, size_t ws_bytes,
                             void* stream) {
  md::EwPlan pl;
  md_status s = md::ew_plan(p, n_atoms, kmax, &pl);
  if (s != MD_OK) return s;
  if (!d_energy || ((uintptr_t)d_energy & 7)) return MD_ERR_INVALID_ARG;
  if (n_atoms > 0 && (!d_pos || !d_charge || !d_force ||
                      (((uintptr_t)d_pos | (uintptr_t)d_charge | (uintptr_t)d_force) & 3)))
    return MD_ERR_INVALID_ARG;
  if (!d_ws || ((uintptr_t)d_ws & 255) || ws_bytes < md::ew_bytes(p, n_atoms, kmax, &pl))
    return MD_ERR_WORKSPACE;
  if (n_atoms >= md::ew_mesh_from(kmax)) {
    md::EwMeshPlan mesh;
    md::ew_mesh_plan(n_atoms, kmax, &mesh);
    return md::launch_ew_mesh(mesh, p, n_atoms, d_pos, d_charge, d_force, d_energy, accumulate ? 1 : 0,
                              d_ws, (hipStream_t)stream) == hipSuccess
               ? MD_OK
               : MD_ERR_HIP;
  }
  md::EwArgs a;
  char* b = (char*)d_ws;
  a.n = n_atoms;
  a.pos = d_pos;
  a.q = d_charge;
  a.force = d_force;
  a.energy = d_energy;
  a.accumulate = accumulate ? 1 : 0;
  a.hdr = (md::WsHeader*)b;
  a.ups = (uint4*)(b + pl.off_ups);
  a.tab = (float2*)(b + pl.off_tab);
  a.parts = (float2*)(b + pl.off_parts);
  a.g = (float2*)(b + pl.off_g);
  a.fpart = (double*)(b + pl.off_parts);
  a.stat = (uint32_t*)(b + pl.off_stat);
  a.splits = pl.splits;
  a.split_rows = pl.split_rows;
  a.erow = (double*)(b + pl.off_erow);
  a.qpart = (double2*)(b + pl.off_qpart);
  a.kx = pl.kx;
  a.ky = pl.ky;
  a.kz = pl.kz;
  a.nzc = pl.nzc;
  a.nzc_pad = pl.nzc_pad;
  a.zblocks = pl.zblocks;
  a.rows = pl.rows;
  a.chunks = pl.chunks;
  a.chunk_atoms = pl.chunk_atoms;
  a.qblocks = pl.qblocks;
  for (int d = 0; d < 3; ++d) a.L[d] = (double)(float)p->box[d];   // the float32 box
  a.alpha = p->ewald_alpha;
  a.coulomb_k = p->coulomb_k;
  hipStream_t st = (hipStream_t)stream;
  unsigned final_blocks = 1;
  if (n_atoms > 0) {
    const unsigned nb = (unsigned)((n_atoms + 255) / 256);
    const unsigned trows = (unsigned)((pl.kx + 1) + (2 * pl.ky + 1) + pl.nzc);
    hipLaunchKernelGGL(md::k_ew_prepare, dim3(nb, trows), dim3(256), 0, st, a);
    hipLaunchKernelGGL(md::k_ew_sf,
                       dim3((unsigned)((pl.rows + md::kEwRows - 1) / md::kEwRows),
                            (unsigned)pl.chunks, (unsigned)pl.zblocks),
                       dim3(1024), 0, st, a);
    hipLaunchKernelGGL(md::k_ew_g, dim3((unsigned)((pl.rows + 3) / 4), (unsigned)pl.zblocks), dim3(256), 0,
                       st, a);
    hipLaunchKernelGGL(md::k_ew_force, dim3((unsigned)((n_atoms + 63) / 64), (unsigned)pl.splits),
                       dim3(256), 0, st, a);
    if (pl.splits > 1) final_blocks += nb;
  } else {
    // no atoms: every term is zero
    a.qblocks = 0;
    a.rows = 0;
  }
  hipLaunchKernelGGL(md::k_ew_final, dim3(final_blocks), dim3(256), 0, st, a);
  return hipGetLastError() == hipSuccess ? MD_OK : MD_ERR_HIP;
}

}  // extern "C"
