// C ABI entry points: argument checks, the cell grid, the workspace carve-up, and
// the launch sequence binning -> pair -> finalize on the caller's stream.
#include <math.h>
#include <string.h>

#include <atomic>
#include <mutex>
#include <utility>

#include "md_common.hpp"

namespace md {

// Workspace of md_forces_f32_noalloc: one per device, held from the library's first use
// on that device until the process ends. Host code reaches it only through the device
// address that hipGetSymbolAddress returns for the current device (noalloc_scratch).
// The array is larger than the size limit on systems by what the limit does not count
// (Plan::uncounted).
constexpr size_t kScratchLimit = (size_t)MD_NOALLOC_MAX_WORKSPACE_BYTES;
constexpr size_t kScratchBytes = kScratchLimit + 65536 + sizeof(long long) * kFsMaxSplit * kFsMaxSlices * kFsMaxCells;
static_assert(sizeof(SysArgs<float>) <= 512, "batch arguments");
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch[kMaxDevices];
static std::mutex g_scratch_mu;

// Device address of the current device's scratch array, looked up once per device.
static md_status noalloc_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return MD_ERR_HIP;
  if (dev < 0 || dev >= kMaxDevices) return MD_ERR_CAPACITY;
  void* ptr = g_scratch[dev].load(std::memory_order_acquire);
  if (!ptr) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    ptr = g_scratch[dev].load(std::memory_order_relaxed);
    if (!ptr) {
      if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr)
        return MD_ERR_HIP;
      g_scratch[dev].store(ptr, std::memory_order_release);
    }
  }
  *out = ptr;
  return MD_OK;
}

// Copies the status word of a workspace to caller memory, in stream order.
__global__ void k_copy_status(const WsHeader* hdr, uint32_t* out) { *out = hdr->status; }

constexpr size_t kArgsOffset = sizeof(WsHeader);   // Plan::off_args

static size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

static md_status check_params(const md_params* p) {
  if (!p) return MD_ERR_INVALID_ARG;
  if (p->n_types < 1) return MD_ERR_INVALID_ARG;
  if (p->n_types > kMaxTypes) return MD_ERR_CAPACITY;
  if (!p->sigma || !p->epsilon) return MD_ERR_INVALID_ARG;
  for (int t = 0; t < p->n_types; ++t) {
    if (!isfinite(p->sigma[t]) || !isfinite(p->epsilon[t]) || p->epsilon[t] < 0)
      return MD_ERR_INVALID_ARG;
  }
  if (!(p->r_cut > 0) || !isfinite(p->r_cut)) return MD_ERR_INVALID_ARG;
  if (!(p->r_switch > 0) || p->r_switch > p->r_cut) return MD_ERR_INVALID_ARG;
  if (!isfinite(p->coulomb_k)) return MD_ERR_INVALID_ARG;
  const uint32_t known = MD_ACCUM_F32_ATOMIC | MD_COULOMB_TRUNCATED | MD_DIAG_COUNTERS |
                         MD_PAIR_PREDICATED | MD_PAIR_FULL_SHELL | MD_PAIR_DRAIN_MASK |
                         MD_COULOMB_EWALD | MD_PAIR_SPLIT_MASK;
  if (p->flags & ~known) return MD_ERR_INVALID_ARG;
  // Ewald's real-space term: a finite positive splitting parameter, on the compacted kernel
  // (float32 sums only there), not together with the truncated form
  if (p->flags & MD_COULOMB_EWALD) {
    if (!(p->ewald_alpha > 0) || !isfinite(p->ewald_alpha)) return MD_ERR_INVALID_ARG;
    if (p->flags & (MD_COULOMB_TRUNCATED | MD_PAIR_PREDICATED)) return MD_ERR_INVALID_ARG;
  }
  // a work split only for the compacted kernel
  if ((p->flags & MD_PAIR_SPLIT_MASK) && (p->flags & MD_PAIR_PREDICATED)) return MD_ERR_INVALID_ARG;
  // another drain depth only for the kernel that has it: the compacted half shell with the
  // whole energy switched (the float64 path is checked in check_call)
  if ((p->flags & MD_PAIR_DRAIN_MASK) &&
      ((p->flags & (MD_ACCUM_F32_ATOMIC | MD_COULOMB_TRUNCATED | MD_PAIR_PREDICATED |
                    MD_PAIR_FULL_SHELL | MD_COULOMB_EWALD)) ||
       !(p->r_switch < p->r_cut)))
    return MD_ERR_INVALID_ARG;
  for (int d = 0; d < 3; ++d)
    if (!isfinite(p->box[d]) || !(p->box[d] > 0)) return MD_ERR_INVALID_ARG;
  return MD_OK;
}

// The compacted pair kernel serves every call except MD_PAIR_PREDICATED and float64 with
// float32 atomics, which take the predicated kernel.
static bool uses_compact(const md_params* p, int real_bytes) {
  return !(p->flags & MD_PAIR_PREDICATED) &&
         !(real_bytes == 8 && (p->flags & MD_ACCUM_F32_ATOMIC));
}

// Split of a home cell's work (FsWork). With fewer cells than compute units the chip is idle
// unless a cell is shared out: parts of the home atoms repeat the staging of the neighbour
// list and its flush, slices of the list repeat the work around each group of home atoms (its
// loads, window searches, partial FIFO passes and sums), and either pays only until there is a
// workgroup per compute unit. The choice is the least time of a model of the kernel in
// microseconds,
//   rounds x (start + loops x (staging of L + groups per wave x (group + filter and force of L)))
// with L the atoms of a slice, fitted to a sweep of 1-8 slices x 1-8 parts (whole calls of
// 3,000 to 92,224 atoms; within 15% over the sweep's faster half, and its choice within 8% of
// the sweep's best). Whole calls, with at most 4 parts and no slices before, and now: 3,000 atoms
// in 8 cells 103 -> 66 us, 9,001 in 40 73 -> 61, 6,000 in 27 68 -> 54, 20,000 in 64 92 -> 82,
// float64 3,000 427 -> 138 (then with 16 waves a workgroup). At 343 and 486 cells (one workgroup each) a second slice
// costs 13% and 30%, so most cells of a grid of more than 256 stay whole. The full shell stores each
// atom's sum without atomics, so its slices stay in one workgroup.
FsWork md_fs_work(uint32_t flags, int real_bytes, int64_t n_cells, int64_t n, bool half) {
  FsWork best{1, 1, 0, 1, 0};
  const uint32_t v = (flags & MD_PAIR_SPLIT_MASK) >> 8;
  if (n > 0 && n_cells > 0 && n_cells <= kFsMaxCells) {
    const bool f64 = real_bytes == 8;
    const double start = f64 ? 13.8 : 11.1, stage = f64 ? 0.0071 : 0.0033, group = f64 ? 10.2 : 9.0,
                 pair = f64 ? 0.0011 : 0.0026, lds = f64 ? 1600 : 3008, wg_waves = f64 ? 8 : 16;
    const double groups = (double)n / (double)n_cells / 4.0;   // of 4 home atoms, per cell
    const double list = (half ? 14.0 : 27.0) * (double)n / (double)n_cells;   // staged atoms
    double t_best = 0;
    for (int s = 1; s <= (half ? kFsMaxSlices : 1); ++s)
      for (int g = 1; g <= kFsMaxSplit; ++g) {
        const double wgs = (double)(n_cells * s * g) / 256.0;
        const double rounds = wgs < 3.0 ? ceil(wgs) : wgs + 0.5;
        const double cut = fmax((double)s, ceil(list / lds)), loops = ceil(cut / s);
        const double waves = groups / g / wg_waves, per_wave = waves < 1.0 ? 1.0 : waves + (f64 ? 0.03 : 0.2);
        const double t =
            rounds * (start + loops * (stage * list / cut + per_wave * (group + pair * list / cut)));
        if (t_best == 0 || t < t_best) {
          t_best = t;
          best.split = g;
          best.slices = s;
        }
      }
  }
  if (v) {
    best.split = v == 1 ? 1 : v == 2 ? 2 : 4;
    return best;
  }
  // The last round of workgroups. What is left of a whole number of them per compute unit goes
  // to the cells that last longest, one more part each; or, where the last round would hold
  // 128 cells or fewer, those cells, the shortest, are cut so that it is a short one. Whole
  // calls without and with: 180 cells 111 -> 86 us, 216 114 -> 95, 448 143 -> 139, 486 165 ->
  // 161, 900 270 -> 262; 264 cells (8 in six parts) 131 -> 108, 300 (44 in three) 145 -> 119, 343
  // (87 in two) 176 -> 150, 630 209 -> 200. From 2048 cells on it is under 1%.
  if (n > 0 && n_cells > 0 && n_cells <= kFsMaxShared) {
    const int64_t units = n_cells * best.split * best.slices, last = units % 256;
    if (last > 128 || (units < 256 && last > 0)) {
      const int64_t more = (256 - last) / best.slices;
      // two half cells of under about 144 atoms take more than one whole (their groups fill the
      // waves worse): 448 cells of 100 atoms 91 us whole, 98 with 64 of them cut
      if (best.split < kFsMaxSplit && (n_cells <= kFsMaxCells || n >= 144 * n_cells)) {
        best.nx = more < n_cells ? more : n_cells;
        best.xsplit = best.split + 1;
        best.xlong = 1;
      }
    } else if (n_cells > kFsMaxCells && last > 0) {
      best.nx = last;
      best.xsplit = last > 66 ? 2 : last < 22 ? 6 : (int)(132 / last);
    }
  }
  return best;
}

static bool half_shell(const md_params* p) {
  return !(p->flags & (MD_ACCUM_F32_ATOMIC | MD_PAIR_FULL_SHELL));
}

// Workgroups of the compacted kernel.
static int64_t fs_units(const md_params* p, const Plan& pl, int64_t n) {
  const FsWork w = md_fs_work(p->flags, pl.real_bytes, pl.n_cells, n, half_shell(p));
  return ((pl.n_cells - w.nx) * w.split + w.nx * w.xsplit) * w.slices;
}

// Grid rule: n_d = floor(L_d / r_cut), one cell fewer when L_d/n_d exceeds r_cut by
// less than 1e-3 A (so rounding of a coordinate at a cell face never hides a pair),
// and at least 2 cells per axis (L >= 2 r_cut keeps the minimum image unique).
md_status make_plan(const md_params* p, int64_t n, int real_bytes, Plan* pl) {
  md_status s = check_params(p);
  if (s != MD_OK) return s;
  if (n < 0) return MD_ERR_INVALID_ARG;
  if (n > kMaxAtoms) return MD_ERR_CAPACITY;
  int64_t cells = 1;
  for (int d = 0; d < 3; ++d) {
    double L = real_bytes == 4 ? (double)(float)p->box[d] : p->box[d];
    double q = floor(L / p->r_cut);
    if (q > 1e7) return MD_ERR_CAPACITY;
    int nd = (int)q;
    if (nd >= 1 && L / nd - p->r_cut < 1e-3) nd -= 1;
    if (nd < 2) return MD_ERR_BOX_TOO_SMALL;
    pl->dims[d] = nd;
    cells *= nd;
    if (cells > kMaxCells) return MD_ERR_CAPACITY;
  }
  pl->n_cells = cells;
  pl->n_tasks = cells * kTasksPerCell;
  pl->n = n;
  pl->real_bytes = real_bytes;
  const size_t nn = (size_t)(n > 0 ? n : 1);
  size_t o = align_up(sizeof(WsHeader));
  static_assert(kArgsOffset % 256 == 0, "alignment");
  pl->off_args = o;      o = align_up(o + sizeof(SysArgs<float>));   // of a batched call
  pl->uncounted = align_up(sizeof(SysArgs<float>));
  pl->off_count = o;     o = align_up(o + sizeof(int32_t) * cells);
  pl->off_start = o;     o = align_up(o + sizeof(int32_t) * (cells + 1));
  pl->off_cell = o;      o = align_up(o + sizeof(int32_t) * nn);
  pl->off_rank = o;      o = align_up(o + sizeof(int32_t) * nn);
  const bool compact = uses_compact(p, real_bytes);
  pl->off_pos = o;       o = align_up(o + (size_t)4 * real_bytes * nn);
  pl->off_hpre = o;      o = align_up(o + (compact ? (size_t)8 * real_bytes * nn : 0));
  pl->off_type = o;      o = align_up(o + sizeof(int32_t) * nn);
  pl->off_perm = o;      o = align_up(o + sizeof(int32_t) * nn);
  // per-atom partials: 27 slots x 3 components for the predicated kernel, or three
  // 64-bit fixed-point sums (float32) or three two-word ones (float64) for the compacted
  // kernel
  pl->off_part = o;
  o = align_up(o + (compact ? sizeof(long long) * 3 * (real_bytes / 4) * nn
                            : (size_t)real_bytes * kSlots * 3 * nn));
  pl->off_facc = o;      o = align_up(o + sizeof(float) * 3 * nn);
  // energy partials: one float64 per task, or one (float64: two) int64 per workgroup of the
  // compacted kernel, as many as any flags could choose. Grids of more than kFsMaxCells cells have
  // fewer, but keep the room of kFsMaxCells, so that a workspace serves a shrinking box
  pl->off_epart = o;
  const size_t task_parts = align_up(sizeof(double) * pl->n_tasks);
  const size_t unit_parts = align_up(sizeof(long long) * (real_bytes / 4) * kFsMaxSplit * kFsMaxSlices *
                                     (cells < kFsMaxCells ? cells : kFsMaxCells));
  o += task_parts > unit_parts ? task_parts : unit_parts;
  if (unit_parts > task_parts) pl->uncounted += unit_parts - task_parts;
  pl->off_lj = o;        o = align_up(o + (size_t)real_bytes * 2 * kMaxTypes * kMaxTypes);
  pl->off_paircount = o; o = align_up(o + sizeof(int32_t) * 2 * nn);
  // binning with per-block LDS histograms when the grid fits in LDS
  pl->bin_blocks = 0;
  pl->bin_chunk = 0;
  if (n > 0 && cells <= kBinLdsCells) {
    int64_t chunk = (n + kBinMaxBlocks - 1) / kBinMaxBlocks;
    chunk = (chunk + kBinChunkUnit - 1) / kBinChunkUnit * kBinChunkUnit;
    pl->bin_chunk = chunk;
    pl->bin_blocks = (int)((n + chunk - 1) / chunk);
  }
  pl->off_bhist = o;     o = align_up(o + sizeof(int32_t) * (size_t)pl->bin_blocks * (cells + 1));
  pl->off_bstat = o;     o = align_up(o + sizeof(uint32_t) * (size_t)(pl->bin_blocks + 1));
  pl->off_order = o;     o = align_up(o + sizeof(int32_t) * cells);
  pl->off_cost = o;      o = align_up(o + sizeof(uint32_t) * cells);
  pl->off_zsplit = o;    o = align_up(o + sizeof(int32_t) * cells);
  pl->off_ukey = o;      o = align_up(o + sizeof(UKey) * nn);
  pl->off_upos = o;      o = align_up(o + (size_t)4 * real_bytes * nn);
  // kinetic-energy partials of two steps (the second set is not counted)
  const size_t ke_bytes = align_up(sizeof(double) * (size_t)ke_blocks(n));
  pl->off_kpart = o;     o += 2 * ke_bytes;
  pl->uncounted += ke_bytes;
  pl->total = o;
  return MD_OK;
}

template <typename Real>
SysArgs<Real> make_args(const md_params* p, const Plan& pl, int64_t n, const Real* pos,
                        const int32_t* type, const Real* q, Real* force, double* energy,
                        void* ws) {
  SysArgs<Real> a;
  char* b = (char*)ws;
  a.pos_in = pos;
  a.type_in = type;
  a.q_in = q;
  a.force_out = force;
  a.energy_out = energy;
  a.hdr = (WsHeader*)b;
  a.count = (int32_t*)(b + pl.off_count);
  a.start = (int32_t*)(b + pl.off_start);
  a.cell = (int32_t*)(b + pl.off_cell);
  a.rank = (int32_t*)(b + pl.off_rank);
  a.pos = (P4<Real>*)(b + pl.off_pos);
  a.hpre = (P4<Real>*)(b + pl.off_hpre);
  a.type = (int32_t*)(b + pl.off_type);
  a.perm = (int32_t*)(b + pl.off_perm);
  a.part = (Real*)(b + pl.off_part);
  a.facc = (float*)(b + pl.off_facc);
  a.epart = (double*)(b + pl.off_epart);
  a.lj = (Real*)(b + pl.off_lj);
  a.paircount = (int32_t*)(b + pl.off_paircount);
  a.acc64 = (long long*)(b + pl.off_part);   // the compacted kernel reuses the partial buffer
  a.bhist = (int32_t*)(b + pl.off_bhist);
  a.bstat = (uint32_t*)(b + pl.off_bstat);
  a.order = (int32_t*)(b + pl.off_order);
  a.cost = (uint32_t*)(b + pl.off_cost);
  a.zsplit = (int32_t*)(b + pl.off_zsplit);
  a.ukey = (UKey*)(b + pl.off_ukey);
  a.upos = (P4<Real>*)(b + pl.off_upos);
  a.bin_blocks = pl.bin_blocks;
  a.bin_chunk = pl.bin_chunk;
  a.n = n;
  a.n_cells = pl.n_cells;
  a.n_tasks = pl.n_tasks;
  a.nx = pl.dims[0];
  a.ny = pl.dims[1];
  a.nz = pl.dims[2];
  a.n_types = p->n_types;
  for (int d = 0; d < 3; ++d) {
    a.L[d] = (Real)p->box[d];
    a.inv_w[d] = (Real)((double)pl.dims[d] / (double)a.L[d]);
  }
  const double rc2 = p->r_cut * p->r_cut, rs2 = p->r_switch * p->r_switch;
  a.rc2 = (Real)rc2;
  a.rs2 = (Real)rs2;
  a.inv_sw = p->r_switch < p->r_cut ? (Real)(1.0 / (rc2 - rs2)) : Real(0);
  a.coulomb_k = (Real)p->coulomb_k;
  // float32: at most 1e17 / r_cut, where erfc(alpha r) is 0 for every distance that counts, so that
  // (alpha r)^2 stays finite
  double alpha = (p->flags & MD_COULOMB_EWALD) ? p->ewald_alpha : 0.0;
  if (sizeof(Real) == 4) alpha = fmin(alpha, 1e17 / p->r_cut);
  a.ewald_alpha = (Real)alpha;
  a.flags = p->flags;
  a.compact = uses_compact(p, (int)sizeof(Real)) ? 1 : 0;
  a.half_shell = a.compact && half_shell(p) ? 1 : 0;
  const FsWork fw = a.compact ? md_fs_work(p->flags, (int)sizeof(Real), pl.n_cells, n, a.half_shell != 0)
                              : FsWork{1, 1, 0, 1, 0};
  a.fs_nx = fw.nx;
  a.fs_xlong = fw.xlong;
  a.fs_xsplit = fw.xsplit;
  a.fs_split = fw.split;
  a.own_nx = fw.nx;
  a.own_xsplit = fw.xsplit;
  a.own_split = fw.split;
  a.fs_slices = a.fs_su = fw.slices;
  a.fs_parts = fs_workgroups(a);
  return a;
}

template SysArgs<float> make_args<float>(const md_params*, const Plan&, int64_t, const float*,
                                         const int32_t*, const float*, float*, double*, void*);
template SysArgs<double> make_args<double>(const md_params*, const Plan&, int64_t,
                                           const double*, const int32_t*, const double*,
                                           double*, double*, void*);

// Synchronous argument checks of one force call; fills the plan.
template <typename Real>
static md_status check_call(const md_params* p, int64_t n, const Real* pos, const int32_t* type,
                            const Real* q, const Real* force, const double* energy,
                            const void* ws, size_t ws_bytes, Plan* pl) {
  md_status s = make_plan(p, n, (int)sizeof(Real), pl);
  if (s != MD_OK) return s;
  if (sizeof(Real) == 8 && (p->flags & MD_PAIR_DRAIN_MASK)) return MD_ERR_INVALID_ARG;
  // float64 with float32 atomics takes the predicated kernel, which has no Ewald form
  if (sizeof(Real) == 8 && (p->flags & MD_COULOMB_EWALD) && (p->flags & MD_ACCUM_F32_ATOMIC))
    return MD_ERR_INVALID_ARG;
  if (!energy || ((uintptr_t)energy & 7)) return MD_ERR_INVALID_ARG;
  if (n > 0) {
    if (!pos || !type || !q || !force) return MD_ERR_INVALID_ARG;
    if (((uintptr_t)pos | (uintptr_t)q | (uintptr_t)force) & (sizeof(Real) - 1))
      return MD_ERR_INVALID_ARG;
    if ((uintptr_t)type & 3) return MD_ERR_INVALID_ARG;
  }
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < pl->total) return MD_ERR_WORKSPACE;
  return MD_OK;
}

// Systems that may share one batched launch: same flags and the same type table.
static bool same_kind(const md_params* x, const md_params* y) {
  if (x->flags != y->flags || x->n_types != y->n_types || x->r_cut != y->r_cut ||
      x->r_switch != y->r_switch || x->coulomb_k != y->coulomb_k ||
      ((x->flags & MD_COULOMB_EWALD) && x->ewald_alpha != y->ewald_alpha))
    return false;
  for (int t = 0; t < x->n_types; ++t)
    if (x->sigma[t] != y->sigma[t] || x->epsilon[t] != y->epsilon[t]) return false;
  return true;
}

// Work units of the systems of one batched launch. A system alone may split its cells to fill
// the chip; in a batch the others fill it, and a split only repeats staging. Each system
// keeps as many workgroups per cell as leave none of them longer than a 512th of the batch's
// work (two per compute unit), at most its own choice; its slices (which fix the results'
// bits) stay, taken in turn by fewer workgroups, and so do its parts, whole ones dealt to fewer
// workgroups (fs_unit): a share of a neighbour's sum then has a bound that a system accepted alone
// keeps (kAccRange). Against parts of a new split: 2 systems of 9,001 atoms 90.8 -> 88.1 us, 4
// 139.3 -> 133.1, 4 of 3,000 105.4 -> 100.8, 6 of 6,000 134.0 -> 136.2, 16 of 2,000 to 200,000 1059.6 ->
// 1061.8. A cell's cost is about its atoms squared plus the staging and group overhead. Systems with
// the costliest workgroups come first, so that short ones fill the tail.
static void batch_units(int n, SysArgs<float>* sys) {
  if (n == 1) return;
  double cost[kBatchMax], total = 0;
  for (int s = 0; s < n; ++s) {
    const double m = (double)sys[s].n / (double)sys[s].n_cells;
    cost[s] = m * m + 60.0 * m;
    total += cost[s] * (double)sys[s].n_cells;
  }
  for (int s = 0; s < n; ++s) {
    SysArgs<float>& a = sys[s];
    if (!(a.flags & MD_PAIR_SPLIT_MASK)) {   // a split that the caller forces stays
      const int units = (int)fmin(64.0, ceil(cost[s] * 512.0 / total));
      a.fs_su = units < a.fs_su ? units : a.fs_su;
      int split = (units + a.fs_su - 1) / a.fs_su;
      split = split < a.own_split ? split : a.own_split;
      // fewer parts where they are as long (of 6 own parts 3 pairs, not 2 pairs and 2 single ones)
      const int most = (a.own_split + split - 1) / split;
      a.fs_split = (a.own_split + most - 1) / most;
      if (a.fs_split < a.own_split || split == 1) a.fs_nx = 0;   // otherwise its own choice as it is
    }
    cost[s] /= (double)(a.fs_su * a.fs_split);
  }
  for (int i = 1; i < n; ++i)   // insertion sort, longest workgroups first
    for (int k = i; k > 0 && cost[k] > cost[k - 1]; --k) {
      std::swap(cost[k], cost[k - 1]);
      std::swap(sys[k], sys[k - 1]);
    }
}

// Copies the systems' arguments to their places in device memory.
__global__ __launch_bounds__(128) void k_put_args(PutArgs p) {
  constexpr int kWords = (int)(sizeof(SysArgs<float>) / 4);
  static_assert(kWords <= 128 && sizeof(SysArgs<float>) % 4 == 0, "a word per thread");
  const int t = threadIdx.x, s = blockIdx.x;
  if (t < kWords)
    reinterpret_cast<uint32_t*>(p.dst[s])[t] = reinterpret_cast<const uint32_t*>(&p.sys[s])[t];
}

static md_status launch_batch(int n, SysArgs<float>* sys, const md_params* p, hipStream_t st) {
  if (n == 0) return MD_OK;
  batch_units(n, sys);
  Batch b;
  b.n = n;
  for (int s = 0; s < kBatchMax; ++s)
    b.sys[s] = reinterpret_cast<const SysArgs<float>*>((char*)sys[s < n ? s : 0].hdr + kArgsOffset);
  for (int s0 = 0; s0 < n; s0 += kPutMax) {
    PutArgs pa;
    pa.n = n - s0 < kPutMax ? n - s0 : kPutMax;
    for (int k = 0; k < kPutMax; ++k) {
      const int s = k < pa.n ? s0 + k : s0;
      pa.dst[k] = const_cast<SysArgs<float>*>(b.sys[s]);
      pa.sys[k] = sys[s];
    }
    hipLaunchKernelGGL(k_put_args, dim3((unsigned)pa.n), dim3(128), 0, st, pa);
  }
  if (launch_binning_batch(b, sys, make_type_table(p), st) != hipSuccess) return MD_ERR_HIP;
  if (launch_pair_fs_batch(b, sys, st) != hipSuccess) return MD_ERR_HIP;
  if (launch_finalize_batch(b, sys, st) != hipSuccess) return MD_ERR_HIP;
  return MD_OK;
}

template <typename Real>
static md_status forces_impl(const md_params* p, int64_t n, const Real* pos,
                             const int32_t* type, const Real* q, Real* force, double* energy,
                             void* ws, size_t ws_bytes, void* stream,
                             uint32_t stages = MD_STAGE_ALL) {
  if (stages & ~(uint32_t)MD_STAGE_ALL) return MD_ERR_INVALID_ARG;
  Plan pl;
  md_status s = check_call<Real>(p, n, pos, type, q, force, energy, ws, ws_bytes, &pl);
  if (s != MD_OK) return s;
  SysArgs<Real> a = make_args<Real>(p, pl, n, pos, type, q, force, energy, ws);
  hipStream_t st = (hipStream_t)stream;
  if ((stages & MD_STAGE_BIN) && launch_binning<Real>(a, make_type_table(p), st) != hipSuccess)
    return MD_ERR_HIP;
  if ((stages & MD_STAGE_PAIR) && launch_pair<Real>(a, st) != hipSuccess) return MD_ERR_HIP;
  if ((stages & MD_STAGE_FINALIZE) && launch_finalize<Real>(a, st) != hipSuccess)
    return MD_ERR_HIP;
  return MD_OK;
}

}  // namespace md

extern "C" {

size_t md_workspace_bytes(const md_params* p, int64_t n_atoms, int double_precision) {
  md::Plan pl;
  if (md::make_plan(p, n_atoms, double_precision ? 8 : 4, &pl) != MD_OK) return 0;
  return pl.total;
}

md_status md_workspace_layout(const md_params* p, int64_t n_atoms, int double_precision,
                              md_layout* out) {
  if (!out) return MD_ERR_INVALID_ARG;
  md::Plan pl;
  md_status s = md::make_plan(p, n_atoms, double_precision ? 8 : 4, &pl);
  if (s != MD_OK) return s;
  for (int d = 0; d < 3; ++d) out->dims[d] = pl.dims[d];
  out->n_cells = pl.n_cells;
  out->cell_start = pl.off_start;
  out->perm = pl.off_perm;
  out->pair_count = pl.off_paircount;
  out->energy_partials = pl.off_epart;
  out->n_energy_partials =
      md::uses_compact(p, double_precision ? 8 : 4)
          ? md::fs_units(p, pl, n_atoms)
          : pl.n_tasks;
  out->z_split = pl.off_zsplit;
  out->total_bytes = pl.total;
  return MD_OK;
}

md_status md_forces_f32(const md_params* p, int64_t n_atoms, const float* d_pos,
                        const int32_t* d_type, const float* d_charge, float* d_force,
                        double* d_energy, void* d_ws, size_t ws_bytes, void* stream) {
  return md::forces_impl<float>(p, n_atoms, d_pos, d_type, d_charge, d_force, d_energy, d_ws,
                                ws_bytes, stream);
}

md_status md_forces_f32_stages(const md_params* p, int64_t n_atoms, const float* d_pos,
                               const int32_t* d_type, const float* d_charge, float* d_force,
                               double* d_energy, void* d_ws, size_t ws_bytes, uint32_t stages,
                               void* stream) {
  return md::forces_impl<float>(p, n_atoms, d_pos, d_type, d_charge, d_force, d_energy, d_ws,
                                ws_bytes, stream, stages);
}

md_status md_forces_f64(const md_params* p, int64_t n_atoms, const double* d_pos,
                        const int32_t* d_type, const double* d_charge, double* d_force,
                        double* d_energy, void* d_ws, size_t ws_bytes, void* stream) {
  return md::forces_impl<double>(p, n_atoms, d_pos, d_type, d_charge, d_force, d_energy, d_ws,
                                 ws_bytes, stream);
}

md_status md_forces_f32_noalloc(const md_params* p, int64_t n_atoms, const float* d_pos,
                                const int32_t* d_type, const float* d_charge, float* d_force,
                                double* d_energy, uint32_t* d_status, void* stream) {
  md::Plan pl;
  // every argument check, the size limit included, before any HIP call
  md_status s = md::make_plan(p, n_atoms, 4, &pl);
  if (s != MD_OK) return s;
  if (pl.total - pl.uncounted > md::kScratchLimit) return MD_ERR_CAPACITY;
  if (d_status && ((uintptr_t)d_status & 3)) return MD_ERR_INVALID_ARG;
  // pointer checks of md_forces_f32 (the workspace is checked against a stand-in with the
  // scratch array's size and alignment)
  s = md::check_call<float>(p, n_atoms, d_pos, d_type, d_charge, d_force, d_energy,
                            (const void*)(uintptr_t)256, md::kScratchBytes, &pl);
  if (s != MD_OK) return s;
  void* ws = nullptr;
  s = md::noalloc_scratch(&ws);
  if (s != MD_OK) return s;
  s = md::forces_impl<float>(p, n_atoms, d_pos, d_type, d_charge, d_force, d_energy, ws,
                             md::kScratchBytes, stream);
  if (s != MD_OK || !d_status) return s;
  hipLaunchKernelGGL(md::k_copy_status, dim3(1), dim3(1), 0, (hipStream_t)stream,
                     (const md::WsHeader*)ws, d_status);
  return hipGetLastError() == hipSuccess ? MD_OK : MD_ERR_HIP;
}

md_status md_run_vv_f32(const md_params* p, int64_t n_atoms, float* d_pos, float* d_vel,
                        const int32_t* d_type, const float* d_charge, const float* d_inv_mass,
                        float* d_force, double dt_fs, int32_t n_steps, double* d_energies,
                        void* d_ws, size_t ws_bytes, void* stream) {
  if (n_steps < 0 || !isfinite(dt_fs)) return MD_ERR_INVALID_ARG;
  md::Plan pl;
  md_status s = md::check_call<float>(p, n_atoms, d_pos, d_type, d_charge, d_force, d_energies,
                                      d_ws, ws_bytes, &pl);
  if (s != MD_OK) return s;
  if (n_atoms > 0 && (!d_vel || !d_inv_mass || (((uintptr_t)d_vel | (uintptr_t)d_inv_mass) & 3)))
    return MD_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  // the box rounded once to float32, as the force path has it
  const float L[3] = {(float)p->box[0], (float)p->box[1], (float)p->box[2]};
  const float dt = (float)dt_fs, h = (float)(0.5 * dt_fs);
  const int64_t kb = (int64_t)(md::align_up(sizeof(double) * (size_t)md::ke_blocks(n_atoms)) / sizeof(double));
  double* kpart = (double*)((char*)d_ws + pl.off_kpart);   // [2][kb], by the step's parity
  if (n_steps > 0 && md::launch_vv_kick_drift(n_atoms, d_pos, d_vel, d_force, d_inv_mass, h, dt, L,
                                              st) != hipSuccess)
    return MD_ERR_HIP;
  // up to 131,072 atoms (between 92,224, 1.7% faster, and 300,000, 0.8% slower) the force
  // path's last kernel moves the atoms
  const bool fused = n_atoms <= 131072;
  const uint32_t stages = fused ? MD_STAGE_BIN | MD_STAGE_PAIR : (uint32_t)MD_STAGE_ALL;
  for (int32_t k = 0; k < n_steps; ++k) {
    s = md::forces_impl<float>(p, n_atoms, d_pos, d_type, d_charge, d_force, d_energies + 2 * k,
                               d_ws, ws_bytes, stream, stages);
    if (s != MD_OK) return s;
    md::VvArgs v;
    v.pos = d_pos;
    v.vel = d_vel;
    v.inv_mass = d_inv_mass;
    v.h = h;
    v.dt = dt;
    for (int d = 0; d < 3; ++d) v.L[d] = L[d];
    v.drift = k + 1 < n_steps;
    v.kpart = kpart + (k & 1) * kb;
    v.kpart_prev = kpart + ((k + 1) & 1) * kb;
    v.ke_prev = k > 0 && n_atoms > 0 ? d_energies + 2 * k - 1 : nullptr;
    if (fused) {
      const md::SysArgs<float> a = md::make_args<float>(p, pl, n_atoms, d_pos, d_type, d_charge,
                                                        d_force, d_energies + 2 * k, d_ws);
      if (md::launch_finalize_vv(a, v, st) != hipSuccess) return MD_ERR_HIP;
    } else if (md::launch_vv_update(n_atoms, d_force, v, st) != hipSuccess) {
      return MD_ERR_HIP;
    }
    if ((n_atoms == 0 || k + 1 == n_steps) &&
        md::launch_ke_sum(n_atoms, v.kpart, d_energies + 2 * k + 1, st) != hipSuccess)
      return MD_ERR_HIP;
  }
  return MD_OK;
}

md_status md_forces_batched(const md_system* sys, int32_t n_sys, void* stream) {
  if (n_sys < 0 || (n_sys > 0 && !sys)) return MD_ERR_INVALID_ARG;
  for (int32_t k = 0; k < n_sys; ++k) {
    md::Plan pl;
    md_status s = md::check_call<float>(&sys[k].p, sys[k].n_atoms, sys[k].d_pos, sys[k].d_type,
                                        sys[k].d_charge, sys[k].d_force, sys[k].d_energy,
                                        sys[k].d_ws, sys[k].ws_bytes, &pl);
    if (s != MD_OK) return s;
  }
  // Systems binned through LDS histograms and forced by the compacted kernel go in
  // batches of up to kBatchMax systems of one kind, in input order; any other system is
  // evaluated on its own.
  hipStream_t st = (hipStream_t)stream;
  md::SysArgs<float> sys_args[md::kBatchMax];
  int n_batch = 0;
  const md_params* kind = nullptr;
  for (int32_t k = 0; k < n_sys; ++k) {
    md::Plan pl;
    md::make_plan(&sys[k].p, sys[k].n_atoms, 4, &pl);
    const bool batchable = sys[k].n_atoms > 0 && pl.bin_blocks > 0 &&
                           !(sys[k].p.flags & MD_PAIR_PREDICATED);
    if (!batchable) {
      md_status s = md_forces_f32(&sys[k].p, sys[k].n_atoms, sys[k].d_pos, sys[k].d_type,
                                  sys[k].d_charge, sys[k].d_force, sys[k].d_energy, sys[k].d_ws,
                                  sys[k].ws_bytes, stream);
      if (s != MD_OK) return s;
      continue;
    }
    if (n_batch == md::kBatchMax || (n_batch > 0 && !md::same_kind(kind, &sys[k].p))) {
      md_status s = md::launch_batch(n_batch, sys_args, kind, st);
      if (s != MD_OK) return s;
      n_batch = 0;
    }
    if (n_batch == 0) kind = &sys[k].p;
    sys_args[n_batch++] = md::make_args<float>(&sys[k].p, pl, sys[k].n_atoms, sys[k].d_pos,
                                        sys[k].d_type, sys[k].d_charge, sys[k].d_force,
                                        sys[k].d_energy, sys[k].d_ws);
  }
  return md::launch_batch(n_batch, sys_args, kind, st);
}

md_status md_read_device_status(const void* d_ws, void* stream, uint32_t* bits) {
  if (!d_ws || !bits) return MD_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  uint32_t v = 0;
  if (hipMemcpyAsync(&v, d_ws, sizeof(v), hipMemcpyDeviceToHost, st) != hipSuccess)
    return MD_ERR_HIP;
  if (hipStreamSynchronize(st) != hipSuccess) return MD_ERR_HIP;
  *bits = v;
  return MD_OK;
}

md_status md_read_diag(const void* d_ws, void* stream, uint64_t counters[5]) {
  if (!d_ws || !counters) return MD_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  md::WsHeader h;
  if (hipMemcpyAsync(&h, d_ws, sizeof(h), hipMemcpyDeviceToHost, st) != hipSuccess)
    return MD_ERR_HIP;
  if (hipStreamSynchronize(st) != hipSuccess) return MD_ERR_HIP;
  for (int k = 0; k < 5; ++k) counters[k] = h.diag[k];
  return MD_OK;
}

md_status md_read_clock(const void* d_ws, void* stream, double* ghz) {
  if (!d_ws || !ghz) return MD_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  md::WsHeader h;
  if (hipMemcpyAsync(&h, d_ws, sizeof(h), hipMemcpyDeviceToHost, st) != hipSuccess)
    return MD_ERR_HIP;
  if (hipStreamSynchronize(st) != hipSuccess) return MD_ERR_HIP;
  *ghz = h.clock[1] ? 0.1 * (double)h.clock[0] / (double)h.clock[1] : 0.0;
  return MD_OK;
}

const char* md_status_string(md_status s) {
  switch (s) {
    case MD_OK: return "ok";
    case MD_ERR_INVALID_ARG: return "invalid argument";
    case MD_ERR_BOX_TOO_SMALL: return "box too small: fewer than 2 cells of edge >= r_cut";
    case MD_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case MD_ERR_HIP: return "HIP runtime error";
    case MD_ERR_DEVICE_STATUS: return "device status word set";
    case MD_ERR_CAPACITY: return "problem exceeds an internal limit";
  }
  return "unknown status";
}

}  // extern "C"
