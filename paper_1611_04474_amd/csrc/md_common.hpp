// Internal declarations shared by the translation units of the force library.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "mdforce.h"

namespace md {

constexpr int kMaxTypes = 64;
constexpr int kTasksPerCell = 14;    // predicated kernel: home cell + 13 forward neighbours
constexpr int kSlots = 27;           // partial-force slots per atom: 14 as home, 13 as neighbour
constexpr int kTile = 256;           // atoms of one cell staged in LDS at a time
constexpr int kPairThreads = 256;    // threads of one predicated pair workgroup (4 waves)
constexpr int64_t kMaxCells = 1 << 24;
constexpr int64_t kMaxAtoms = (int64_t)1 << 30;
constexpr int kBinLdsCells = 32768;  // largest grid binned with a per-block LDS histogram
constexpr int kBinMaxBlocks = 1024;  // blocks of that pass
constexpr int kBinThreads = 512;     // threads per block of that pass
constexpr int kBinChunkUnit = 2048;  // atoms per block: a multiple of this (4 per thread)
// A^2 added to rc^2 by the compacted kernel's expanded-form prefilter (its constants per
// home atom are written by the in-cell sort)
constexpr float kPrefilterMargin = 0.05f;

// Workspace header (first 256 bytes).
// Drain depth selected by MD_PAIR_DRAIN in md_params.flags (2 when the field is 0).
__host__ __device__ inline int md_pair_drain(uint32_t flags) {
  const uint32_t v = (flags & MD_PAIR_DRAIN_MASK) >> 5;
  return v == 0 ? 2 : v == 1 ? 1 : v == 2 ? 3 : 4;
}

// Work units of the compacted pair kernel. The neighbour list of a home cell is cut into
// `slices` equal slices (more where one would not fit the LDS), the cell's groups of home atoms
// into `split` interleaved parts (`xsplit` in nx of the cells: the longest ones or the shortest
// ones of the launch order), and one workgroup takes a slice and a part.
// A home atom's partial force is rounded to fixed point once per slice, so the number of
// slices depends on the grid, the atom count, the precision and the shell (and, where a list
// does not fit the LDS, on what its capacity depends on: types, counters, drain depth), never on the
// split that a caller forces or on the batch a system runs in: those change which workgroup
// does the work and not one bit of the result.
struct FsWork {
  int split;      // parts of a cell's home atoms
  int slices;     // slices of its neighbour list
  int64_t nx;     // cells with another split
  int xsplit;     // theirs
  int xlong;      // 1: they are the first (longest) of the launch order, 0: the last
};
constexpr int kFsMaxSplit = 8, kFsMaxSlices = 8;
constexpr int kFsMaxCells = 256;     // larger grids: one workgroup for most cells unless forced
constexpr int kFsMaxShared = 2048;   // still larger ones: for every cell
FsWork md_fs_work(uint32_t flags, int real_bytes, int64_t n_cells, int64_t n, bool half);

struct WsHeader {
  uint32_t status;
  uint32_t pad0;
  unsigned long long diag[5];   // candidates, filter passes, cutoff passes, filtered slots,
                                // force lanes evaluated
  unsigned long long clock[2];  // compacted pair kernel since the last binning, summed over
                                // its workgroups: shader-clock cycles, 100 MHz ticks
  uint32_t cost_key;            // kCostKey when cost[] holds the last pair kernel's times
  uint32_t cost_cells;          // ... of a grid of this many cells
  uint32_t pad1[46];
};
constexpr uint32_t kCostKey = 0x4d44434fu;
static_assert(sizeof(WsHeader) == 256, "header size");

// An atom's in-cell sort key and type, written by the scatter with one 16-byte store.
struct alignas(16) UKey {
  unsigned long long key;
  int32_t type;
  int32_t pad;
};

template <typename Real>
struct alignas(4 * sizeof(Real)) P4 {
  Real x, y, z, w;
};

// A small non-negative integer carried in a Real slot as bits (no arithmetic is done on it).
template <typename Real>
__device__ inline Real int_to_slot(int32_t v) {
  if constexpr (sizeof(Real) == 4) return __int_as_float(v);
  else return __longlong_as_double((long long)v);
}
template <typename Real>
__device__ inline int32_t slot_to_int(Real v) {
  if constexpr (sizeof(Real) == 4) return __float_as_int(v);
  else return (int32_t)__double_as_longlong(v);
}

// Cell grid and workspace carve-up for one system.
struct Plan {
  int32_t dims[3];
  int64_t n_cells;
  int64_t n_tasks;
  int64_t n;
  int real_bytes;               // 4 or 8
  // byte offsets
  size_t off_args, off_count, off_start, off_cell, off_rank, off_pos, off_hpre, off_type, off_perm,
      off_part, off_facc, off_epart, off_lj, off_paircount, off_bhist, off_bstat, off_order,
      off_cost,
      off_zsplit, off_ukey, off_upos, off_kpart, total;
  size_t uncounted;             // bytes that the no-allocation call's limit does not count: the
                                // batch arguments, the energy partials beyond one word per task, and
                                // the second set of kinetic-energy partials
  int bin_blocks;               // blocks of the LDS-histogram binning pass (0: global atomics)
  int64_t bin_chunk;            // atoms per such block
};

// Computes the grid and workspace layout; returns MD_OK or an error code.
md_status make_plan(const md_params* p, int64_t n, int real_bytes, Plan* out);

// Kernel-side constants of one system.
template <typename Real>
struct SysArgs {
  // inputs
  const Real* pos_in;          // [n][3]
  const int32_t* type_in;      // [n]
  const Real* q_in;            // [n]
  Real* force_out;             // [n][3]
  double* energy_out;          // [1]
  // workspace
  WsHeader* hdr;
  int32_t* count;              // [n_cells]
  int32_t* start;              // [n_cells+1]
  int32_t* cell;               // [n]
  int32_t* rank;               // [n] (also the in-cell sort's member list of a cell of more
                               // than 1024 atoms, with the fused scan)
  UKey* ukey;                  // [n] in-cell sort keys and types, in cell order before the
                               // in-cell sort (with the fused scan: in cell order within
                               // each histogram block's range)
  P4<Real>* upos;              // [n] wrapped (x, y, z, q), same order
  P4<Real>* pos;               // [n] sorted (x,y,z,q)
  P4<Real>* hpre;              // [2n] sorted, for the compacted kernel (written by the
                               // in-cell sort): the atom's prefilter constants as a home
                               // atom, (ax, ay, az, thb) = (-2 a, rc^2 + margin - |a|^2 -
                               // 2 a.o) with a = r - o, o its cell's centre, and
                               // (k q, type n_types as integer bits, 0, 0)
  int32_t* type;               // [n] sorted
  int32_t* perm;               // [n] sorted -> original
  Real* part;                  // [kSlots][3][n]
  float* facc;                 // [3][n]
  double* epart;               // [n_tasks]
  Real* lj;                    // [n_types^2][2] (c12, c6)
  int32_t* paircount;          // [2][n]: caller order (after finalize), sorted order (pass)
  long long* acc64;            // per-atom fixed-point sums of the compacted kernel: float32
                               // [3][n] (2^-28 kcal/mol/A); float64 [2][3][n], the high
                               // words (2^-20) then the low words (2^-72)
  int32_t* bhist;              // grids of at most 1024 cells: [bin_blocks][n_cells + 1] each
                               // block's start of every cell within its range (then its
                               // atom count); larger grids: [bin_blocks][n_cells] per-block
                               // cell counts (offsets in place after k_bin_colscan)
  uint32_t* bstat;             // [bin_blocks] per-block status bits
  int32_t* order;              // [n_cells] launch order of the home cells, longest first
  uint32_t* cost;              // [n_cells] each home cell's time in the last pair kernel
  int32_t* zsplit;             // [n_cells] atoms of each cell in its lower z half
  // scalars
  int64_t n, n_cells, n_tasks;
  int bin_blocks;
  int64_t bin_chunk;
  int nx, ny, nz, n_types;
  Real L[3];                   // box (rounded once to Real)
  Real inv_w[3];               // n_d / L_d
  Real rc2, rs2, inv_sw;       // inv_sw = 1/(rc2 - rs2), 0 when switching is off
  Real coulomb_k;
  Real ewald_alpha;            // 1/A, with MD_COULOMB_EWALD (0 otherwise)
  uint32_t flags;
  int compact;                 // 1: per-atom sums come from the compacted pair kernel (acc64,
                               //    or, float32 only, facc with MD_ACCUM_F32_ATOMIC)
  int half_shell;              // 1: the compacted kernel visits each pair once and adds
                               //    into acc64 with integer atomics (acc64 starts at zero)
  int64_t fs_parts;            // energy partials of a call on its own (a batched one may write fewer)
  int64_t fs_nx;               // FsWork: cells of the other split, which ends of the launch
  int fs_xlong, fs_xsplit;     // order, and that split
  int fs_split;                // parts of the other cells' home atoms, a workgroup each
  int fs_slices;               // slices of its neighbour list, at least (FsWork)
  int fs_su;                   // slices spread over workgroups (fs_slices, or fewer in a batch
                               // that fills the chip: then a workgroup takes several in turn)
  // fs_nx, fs_xsplit and fs_split of a call of its own: in a batch fs_split parts are made of
  // these (see fs_unit)
  int64_t own_nx;
  int own_xsplit, own_split;
};

// Workgroups of the compacted kernel for one system.
template <typename Real>
__host__ __device__ inline int64_t fs_workgroups(const SysArgs<Real>& a) {
  return ((a.n_cells - a.fs_nx) * a.fs_split + a.fs_nx * a.fs_xsplit) * a.fs_su;
}

// Up to kBatchMax systems evaluated by one launch of each kernel of the path. Their
// arguments (about 380 bytes each) stand in device memory, in each system's workspace, put
// there by k_put_args; the kernels get the systems' block ranges and the arguments'
// addresses. Block b of a batched launch belongs to the system s with cum[s] <= b < cum[s+1],
// as its local block b - cum[s]. Handed over by value instead, ten systems fill the 4 KB of
// kernel arguments, and a larger batch takes another launch of each kernel: 16 requests of 2k-200k
// atoms 1148 us that way, 1130 this way.
constexpr int kBatchMax = 128;
constexpr int kPutMax = 10;     // systems per k_put_args launch (kernel arguments under 4 KB)

struct Batch {
  int n;
  int64_t cum[kBatchMax + 1];
  const SysArgs<float>* sys[kBatchMax];
};

struct PutArgs {
  int n;
  SysArgs<float>* dst[kPutMax];
  SysArgs<float> sys[kPutMax];
};
static_assert(sizeof(Batch) + sizeof(double) * 2 * kMaxTypes <= 4096 - 64, "kernel arguments");
static_assert(sizeof(PutArgs) <= 4096 - 64, "kernel arguments");

// The system of block b and its local block: lane l compares the ends of systems l and
// l + 64 with b, so that the table is read in one round trip.
__device__ inline const SysArgs<float>* batch_pick(const Batch& t, int64_t b, int64_t& local) {
  static_assert(kBatchMax == 128, "two table entries per lane");
  const int lane = threadIdx.x & 63;
  const int64_t e0 = t.cum[lane + 1], e1 = t.cum[lane + 65];   // past n: at least cum[n]
  const int s = __builtin_popcountll(__builtin_amdgcn_ballot_w64(e0 <= b)) +
                __builtin_popcountll(__builtin_amdgcn_ballot_w64(e1 <= b));
  local = b - t.cum[s];
  return t.sys[s];
}

// A system's arguments, read through the scalar cache; its pointers are to global memory.
__device__ inline SysArgs<float> batch_args(const SysArgs<float>* p) {
  typedef const __attribute__((address_space(4))) SysArgs<float>* cptr;
  SysArgs<float> a;
  __builtin_memcpy(&a, (cptr)(uintptr_t)p, sizeof(a));
  auto global = [](auto& q) {
    typedef std::remove_reference_t<decltype(*q)> T;
    q = (T*)(__attribute__((address_space(1))) T*)q;
  };
  global(a.pos_in); global(a.type_in); global(a.q_in); global(a.force_out); global(a.energy_out);
  global(a.hdr); global(a.count); global(a.start); global(a.cell); global(a.rank);
  global(a.ukey); global(a.upos); global(a.pos); global(a.hpre); global(a.type); global(a.perm);
  global(a.part); global(a.facc); global(a.epart); global(a.lj); global(a.paircount);
  global(a.acc64); global(a.bhist); global(a.bstat); global(a.order); global(a.cost);
  global(a.zsplit);
  return a;
}

// Per-type sigma and epsilon, mixed into the LJ table by the binning stage.
struct TypeTable {
  double sigma[kMaxTypes];
  double eps[kMaxTypes];
};

template <typename Real>
SysArgs<Real> make_args(const md_params* p, const Plan& pl, int64_t n, const Real* pos,
                        const int32_t* type, const Real* q, Real* force, double* energy,
                        void* ws);

// Launchers (each enqueues on `stream`, returns hipSuccess or an error).
TypeTable make_type_table(const md_params* p);
template <typename Real>
hipError_t launch_binning(const SysArgs<Real>& a, const TypeTable& tt, hipStream_t stream);
template <typename Real>
hipError_t launch_pair(const SysArgs<Real>& a, hipStream_t stream);
template <typename Real>
hipError_t launch_finalize(const SysArgs<Real>& a, hipStream_t stream);
template <typename Real>
hipError_t launch_pair_fs(const SysArgs<Real>& a, hipStream_t stream);

// Batched float32 launchers over n systems' arguments (host copies; b.sys holds the addresses
// of the device copies). Every system of the batch has n > 0, uses the LDS-histogram binning
// (bin_blocks > 0), the compacted kernel, and the same flags and type table.
hipError_t launch_binning_batch(Batch& b, const SysArgs<float>* sys, const TypeTable& tt,
                                hipStream_t stream);
hipError_t launch_pair_fs_batch(Batch& b, const SysArgs<float>* sys, hipStream_t stream);
hipError_t launch_finalize_batch(Batch& b, const SysArgs<float>* sys, hipStream_t stream);

// Sets cum[] of a batch from per-system block counts (entries past the last system repeat
// the total); returns the total.
template <typename F>
inline int64_t batch_blocks(Batch& b, const SysArgs<float>* sys, F per_sys) {
  b.cum[0] = 0;
  for (int s = 0; s < kBatchMax; ++s) b.cum[s + 1] = b.cum[s] + (s < b.n ? per_sys(sys[s]) : 0);
  return b.cum[b.n];
}

// Velocity-Verlet steps of md_run_vv_f32 (md_integrate.hip, md_finalize.hip). kick_drift: v += h
// F/m, x += dt v wrapped into [0, L). finalize_vv: the force path's last kernel with the step's
// second kick and, with drift set, the next step's kick and drift; vv_update: the two kicks and
// the drift alone. The kinetic energies go to per-block partials kpart ([ke_blocks(n)] doubles),
// which the next step's launch (as kpart_prev) or ke_sum sums in a fixed order.
struct VvArgs {
  float *pos, *vel;            // [n][3]
  const float* inv_mass;       // [n]
  float h, dt, L[3];
  int drift;
  double* kpart;
  const double* kpart_prev;
  double* ke_prev;             // null: no previous step
};
__host__ __device__ inline int64_t ke_blocks(int64_t n) { return n > 0 ? (n + 255) / 256 : 1; }
hipError_t launch_vv_kick_drift(int64_t n, float* pos, float* vel, const float* force,
                                const float* inv_mass, float h, float dt, const float* L,
                                hipStream_t stream);
hipError_t launch_finalize_vv(const SysArgs<float>& a, const VvArgs& v, hipStream_t stream);
hipError_t launch_vv_update(int64_t n, const float* force, const VvArgs& v, hipStream_t stream);
hipError_t launch_ke_sum(int64_t n, const double* kpart, double* ke, hipStream_t stream);

}  // namespace md
