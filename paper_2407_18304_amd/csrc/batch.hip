// batch.hip -- one persistent launch over many AMR-like patches, each with its
// own cell count, group count, group edges and opacity table (the patch
// layout of an adaptive mesh, where every patch holds its own SoA block).
//
// Work lists: the patches are cut into items, ordered by decreasing group count
// (the costliest work first, so the tail of the launch is made of cheap items;
// batch_items.hpp).  By default one workgroup runs one item and
// the hardware hands out the items (k_batch_items).  In the other scopes a wave
// or a workgroup takes the next item with one atomic increment of a global
// counter, stages that patch's tables in its LDS slot, sets its lane count per
// cell to the next power of two >= N_g/G, and runs the same per-cell state
// machine as the single-table kernel (cell groups refill from the item's cells
// as their cells finish); a tiny kernel clears the counter before that, so the
// pair can be captured in a hipGraph and replayed.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/mgrhd.h"
#include "batch_infer.hpp"
#include "solver_kernel.hpp"

namespace mgrhd {

constexpr int kBatchNGM = 128;  // group capacity of a wave's LDS table slot

using Item = BatchItem;

struct BatchArgs {
  const KArgs* patches;  // device array, one KArgs per patch
  const Item* items;     // device array
  int32_t* counter;      // device, cleared before each launch
  int64_t n_items;
};

__global__ void k_clear_counter(int32_t* counter) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *counter = 0;
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Stage the tables of one patch into this wave's LDS slot (wave scope).
template <int MODE, int NGM>
__device__ __forceinline__ bool stage_tables_wave(const KArgs& a, Tables<NGM>& t, int lane) {
  if (lane == 0) t.bad = 0;
  wave_sync();
  const int ng = a.ng;
  if (ng > NGM) {
    t.bad = 1;
    wave_sync();
    return false;
  }
  for (int g = lane; g <= ng; g += kWave)
    if (!table_edge<NGM, MODE>(a, t, g)) atomicOr(&t.bad, 1);
  wave_sync();
  for (int g = lane; g < ng; g += kWave)
    if (!table_group<NGM, MODE>(a, t, g)) atomicOr(&t.bad, 1);
  wave_sync();
  return t.bad == 0;
}

// A copy of *p in scalar registers: every lane reads the same words and the
// first lane's value is taken, so the compiler knows the fields are uniform.
template <class T>
__device__ __forceinline__ T load_uniform(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "whole words");
  constexpr int kWords = sizeof(T) / 4;
  int w[kWords];
  const int* src = reinterpret_cast<const int*>(p);
#pragma unroll
  for (int k = 0; k < kWords; ++k) w[k] = __builtin_amdgcn_readfirstlane(src[k]);
  T r;
  __builtin_memcpy(&r, w, sizeof(T));
  return r;
}

// Lanes per cell for N_g groups at G groups per lane: the next power of two
// >= N_g / G.  The state machine is compiled for each.
template <int G, int MODE, int NGM, bool FULL, class LS, class Q>
__device__ __forceinline__ void run_item_lpc(const KArgs& a, const Tables<NGM>& tab,
                                             const LS& ls, int lane, Q q, int lpc) {
  switch (lpc) {
    case 1: run_cells<G, 1, MODE, NGM, false, FULL>(a, tab, ls, lane, q); break;
    case 2: run_cells<G, 2, MODE, NGM, false, FULL>(a, tab, ls, lane, q); break;
    case 4: run_cells<G, 4, MODE, NGM, false, FULL>(a, tab, ls, lane, q); break;
    case 8: run_cells<G, 8, MODE, NGM, false, FULL>(a, tab, ls, lane, q); break;
    case 16: run_cells<G, 16, MODE, NGM, false, FULL>(a, tab, ls, lane, q); break;
    case 32: run_cells<G, 32, MODE, NGM, false, FULL>(a, tab, ls, lane, q); break;
    default:  // a patch wider than 32 lanes of G groups
      if constexpr (G * 32 < NGM) run_cells<G, kWave, MODE, NGM, false, FULL>(a, tab, ls, lane, q);
      break;
  }
}

// TRY_FULL: items whose N_g fills every slot (N_g = lanes per cell x G) run
// the state machine compiled for that case (no per-slot group checks).
template <int G, int MODE, int NGM, bool TRY_FULL, class LS, class Q>
__device__ __forceinline__ void run_item(const KArgs& a, const Tables<NGM>& tab,
                                         const LS& ls_block, int lane, Q q) {
  // a is an entry of the batch's device array of patch arguments
  const LS ls = ls_block.with_args((KArgsRef)&a);
  int lpc = 1;
  while (lpc * G < a.ng) lpc <<= 1;
  if (TRY_FULL && lpc * G == a.ng)
    run_item_lpc<G, MODE, NGM, true>(a, tab, ls, lane, q, lpc);
  else
    run_item_lpc<G, MODE, NGM, false>(a, tab, ls, lane, q, lpc);
}

// 2 groups per lane leave room in LDS for the old-time fluxes and velocity
// (re-reading them from HBM in the outer stage, or a table slot narrower than
// 128 groups to fit a third workgroup per CU, measured slower: the extra
// registers spill); with 4 they are re-read from HBM by the outer stage.
template <int G, int MODE, int NGM>
__global__ __launch_bounds__(kBlock, 2) void k_batch(BatchArgs b) {
  static_assert(G * kWave >= NGM, "a wave holds the widest patch");
  __shared__ Tables<NGM> tabs[kBlock / kWave];
  using LS = LaneStore<G, G == 2, kBlock, true>;  // constants read where used
  __shared__ double lane_lds[LS::kSlots * kBlock];
  __shared__ double cell_lds[LS::kCellWords];
  const LS ls{lane_lds + threadIdx.x, cell_lds, nullptr};  // run_item sets the arguments
  const int lane = threadIdx.x % kWave;
  Tables<NGM>& tab = tabs[threadIdx.x / kWave];
  int cur_patch = -1;
  bool table_ok = false;
  for (;;) {
    // the wave takes the next work item (all lanes are active here)
    int it = 0;
    if (lane == 0) it = atomicAdd(b.counter, 1);
    it = __builtin_amdgcn_readfirstlane(it);
    if (it >= b.n_items) break;
    const Item item = load_uniform(b.items + it);
    const KArgs& a = b.patches[item.patch];
    if (item.patch != cur_patch) {
      table_ok = stage_tables_wave<MODE, NGM>(a, tab, lane);
      cur_patch = item.patch;
    }
    if (!table_ok) {
      for (int64_t i = item.c0 + lane; i < item.c1; i += kWave) {
        copy_through(a, state_ptrs((KArgsRef)&a), i, 0, 1);  // out of place: inputs
        if (a.status) a.status[i] = MGRHD_ST_BAD_TABLE;
        if (a.iters) a.iters[i] = 0;
        if (a.outer) a.outer[i] = 0;
        if (a.trace)
          for (int k = 0; k < a.max_outer; ++k) a.trace[(int64_t)k * a.n + i] = -1;
      }
      continue;
    }
    run_item<G, MODE, NGM, false>(a, tab, ls, lane, WaveRange{item.c0, item.c1});
  }
}

// Items per workgroup: the four waves of a workgroup take one item together,
// share one LDS table slot (so LDS leaves room for 3 workgroups per CU) and
// take the item's cells through an LDS counter, so the cells in flight in a
// workgroup share the cache lines of every SoA row.  Waves that run out of
// cells wait at the item's end for the others.
template <int G, int MODE, int NGM>
__global__ __launch_bounds__(kBlock, 2) void k_batch_wg(BatchArgs b) {
  static_assert(G * kWave >= NGM, "a wave holds the widest patch");
  __shared__ Tables<NGM> tab;
  __shared__ int item_s, taken;
  using LS = LaneStore<G, G == 2, kBlock, true>;  // constants read where used
  __shared__ double lane_lds[LS::kSlots * kBlock];
  __shared__ double cell_lds[LS::kCellWords];
  const LS ls{lane_lds + threadIdx.x, cell_lds, nullptr};  // run_item sets the arguments
  const int lane = threadIdx.x % kWave;
  int cur_patch = -1;
  bool table_ok = false;
  for (;;) {
    if (threadIdx.x == 0) {
      item_s = atomicAdd(b.counter, 1);
      taken = 0;
    }
    __syncthreads();
    const int it = __builtin_amdgcn_readfirstlane(item_s);
    if (it >= b.n_items) break;
    const Item item = load_uniform(b.items + it);
    const KArgs& a = b.patches[item.patch];
    if (item.patch != cur_patch) {  // uniform over the workgroup
      table_ok = stage_tables<NGM, MODE>(a, tab);
      cur_patch = item.patch;
    }
    if (!table_ok) {
      for (int64_t i = item.c0 + threadIdx.x; i < item.c1; i += kBlock) {
        copy_through(a, state_ptrs((KArgsRef)&a), i, 0, 1);  // out of place: inputs
        if (a.status) a.status[i] = MGRHD_ST_BAD_TABLE;
        if (a.iters) a.iters[i] = 0;
        if (a.outer) a.outer[i] = 0;
        if (a.trace)
          for (int k = 0; k < a.max_outer; ++k) a.trace[(int64_t)k * a.n + i] = -1;
      }
    } else {
      run_item<G, MODE, NGM, true>(a, tab, ls, lane, BlockQueue{&taken, item.c0, item.c1});
    }
    __syncthreads();  // the item is done before the next one resets the counter
  }
}

// One workgroup per item (scope 1 at 2 groups per lane), started by the
// hardware as earlier ones end.  The state machine is the single-table
// kernel's for the item's lane count; FULL: every item's N_g fills its lanes,
// which leaves four waves per SIMD (k_source_update).  The patch's constants
// are read where they are used (held in scalar registers they spilled 30 of
// them in each state machine, 1% slower).  LDS is dynamic, as much as the
// largest item of the launch needs.  Bound by the vector ALU as the
// single-table kernel.  Taking items from a counter instead (k_batch_wg) asks
// for an LDS slot for 128 groups, three workgroups per CU, and waits at every
// item's end for the last of its cells: 24 patches of 1.3e6 cells 8.64 -> 8.04
// ms, 12 patches 3.48 -> 2.79 ms, 6 patches of 3e5 cells 1.41 -> 0.57 ms.
template <int G, int LPC, int MODE, bool FULL>
__device__ __forceinline__ void run_item_block(const KArgs& a, KArgsRef ap, const Item& item,
                                               unsigned char* lds) {
  constexpr int kThreads = block_threads<G, FULL, MODE, false>();
  run_block<G, LPC, MODE, false, FULL>(a, ap, item.c0, item.c1,
                                       *(BlockLds<G, LPC, kThreads, true>*)lds);
}

template <int G, int MODE, bool FULL>
__global__ __launch_bounds__((block_threads<G, FULL, MODE, false>()), FULL ? 4 : 3) void k_batch_items(
    const KArgs* patches, const Item* items) {
  extern __shared__ __attribute__((aligned(16))) unsigned char batch_lds[];
  typedef const Item __attribute__((address_space(4)))* ItemRef;
  const ItemRef ip = (ItemRef)(items + blockIdx.x);
  const Item item{ip->patch, 0, ip->c0, ip->c1};
  const KArgsRef ap = (KArgsRef)(patches + item.patch);
  KArgs a;
  __builtin_memcpy(&a, (const KArgs*)ap, sizeof(KArgs));
  if (a.ng <= G)
    run_item_block<G, 1, MODE, FULL>(a, ap, item, batch_lds);
  else if (a.ng <= 2 * G)
    run_item_block<G, 2, MODE, FULL>(a, ap, item, batch_lds);
  else if (a.ng <= 4 * G)
    run_item_block<G, 4, MODE, FULL>(a, ap, item, batch_lds);
  else if (a.ng <= 8 * G)
    run_item_block<G, 8, MODE, FULL>(a, ap, item, batch_lds);
  else if (a.ng <= 16 * G)
    run_item_block<G, 16, MODE, FULL>(a, ap, item, batch_lds);
  else if (a.ng <= 32 * G)
    run_item_block<G, 32, MODE, FULL>(a, ap, item, batch_lds);
  else
    run_item_block<G, 64, MODE, FULL>(a, ap, item, batch_lds);
}

// Threads of a workgroup of k_batch_items (of any mean mode), and its LDS with
// lpc lanes per cell.
template <bool FULL>
constexpr int kItemThreads = block_threads<2, FULL, MGRHD_MEAN_PPL_FREE, false>();
template <bool FULL>
static size_t item_lds(int lpc) {
  switch (lpc) {
    case 1: return sizeof(BlockLds<2, 1, kItemThreads<FULL>>);
    case 2: return sizeof(BlockLds<2, 2, kItemThreads<FULL>>);
    case 4: return sizeof(BlockLds<2, 4, kItemThreads<FULL>>);
    case 8: return sizeof(BlockLds<2, 8, kItemThreads<FULL>>);
    case 16: return sizeof(BlockLds<2, 16, kItemThreads<FULL>>);
    case 32: return sizeof(BlockLds<2, 32, kItemThreads<FULL>>);
    default: return sizeof(BlockLds<2, 64, kItemThreads<FULL>>);
  }
}
static int item_threads(bool full) { return full ? kItemThreads<true> : kItemThreads<false>; }

using ItemsFn = void (*)(const KArgs*, const Item*);
static ItemsFn items_fn(int mode, bool full) {
  static const ItemsFn fn[2][3] = {
      {k_batch_items<2, MGRHD_MEAN_PC, false>, k_batch_items<2, MGRHD_MEAN_PPL_FIXED, false>,
       k_batch_items<2, MGRHD_MEAN_PPL_FREE, false>},
      {k_batch_items<2, MGRHD_MEAN_PC, true>, k_batch_items<2, MGRHD_MEAN_PPL_FIXED, true>,
       k_batch_items<2, MGRHD_MEAN_PPL_FREE, true>}};
  return fn[full ? 1 : 0][mode];
}

using BatchFn = void (*)(BatchArgs);
// the kernel for g groups per lane, mean mode, and items per wave (scope 0) or
// per workgroup (scope 2, and scope 1 at 4 groups per lane)
static BatchFn batch_fn(int g, int mode, int scope) {
  static const BatchFn wave[2][3] = {
      {k_batch<2, MGRHD_MEAN_PC, kBatchNGM>, k_batch<2, MGRHD_MEAN_PPL_FIXED, kBatchNGM>,
       k_batch<2, MGRHD_MEAN_PPL_FREE, kBatchNGM>},
      {k_batch<4, MGRHD_MEAN_PC, kBatchNGM>, k_batch<4, MGRHD_MEAN_PPL_FIXED, kBatchNGM>,
       k_batch<4, MGRHD_MEAN_PPL_FREE, kBatchNGM>}};
  static const BatchFn wg2[2][3] = {
      {k_batch_wg<2, MGRHD_MEAN_PC, kBatchNGM>, k_batch_wg<2, MGRHD_MEAN_PPL_FIXED, kBatchNGM>,
       k_batch_wg<2, MGRHD_MEAN_PPL_FREE, kBatchNGM>},
      {k_batch_wg<4, MGRHD_MEAN_PC, kBatchNGM>, k_batch_wg<4, MGRHD_MEAN_PPL_FIXED, kBatchNGM>,
       k_batch_wg<4, MGRHD_MEAN_PPL_FREE, kBatchNGM>}};
  const int gi = g == 4 ? 1 : 0;
  if (scope == 0) return wave[gi][mode];
  return wg2[gi][mode];
}

}  // namespace mgrhd

using namespace mgrhd;

struct mgrhd_batch {
  int32_t n_patches = 0;
  int32_t mode = 0;
  int64_t n_cells = 0;
  int32_t max_groups = 0;
  KArgs* d_patches = nullptr;
  int32_t* d_counter = nullptr;
  std::vector<KArgs> h_patches;
  // tuning
  int32_t groups_per_lane = 2;
  int32_t scope = 1;          // 0: items per wave, 1 | 2: items per workgroup
  int32_t blocks_per_cu = 0;  // 0 = all resident
  int64_t chunk = 256;
  // The two work lists, rebuilt when `chunk` changes and only then: a graph of
  // the caller's that ran the batch reads the list of the scope it was captured
  // in, whatever scope is set later.
  bool items_dirty = true;
  Item* d_items = nullptr;    // by cells (counter scopes, inference)
  int64_t n_items = 0;
  std::vector<std::pair<int32_t, std::pair<int64_t, int64_t>>> ng_items;
  Item* d_rounds = nullptr;   // by rounds (k_batch_items), the full ones first
  int64_t n_rounds = 0, n_full = 0;
  size_t lds_full = 0, lds_rest = 0;  // most LDS that a full item takes, and another
  // warm-start networks attached per group count (inference enqueued before
  // the solve)
  struct Net {
    int32_t ng;
    mgrhd_mlp* m;
    const float *x_mean, *x_istd, *y_mean, *y_std;
  };
  std::vector<Net> nets;
  int32_t guess_kind = 0;
  // graph
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

static int device_cus() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus < 1)
    cus = 256;
  return cus;
}

static int upload_items(const std::vector<Item>& items, Item*& d) {
  if (d) (void)hipFree(d);
  d = nullptr;
  if (items.empty()) return 0;
  const size_t bytes = sizeof(Item) * items.size();
  return hipMalloc(&d, bytes) == hipSuccess &&
                 hipMemcpy(d, items.data(), bytes, hipMemcpyHostToDevice) == hipSuccess
             ? 0 : MGRHD_E_DEVICE;
}

static std::vector<PatchSize> patch_sizes(const mgrhd_batch* bt) {
  std::vector<PatchSize> sizes;
  for (const KArgs& a : bt->h_patches) sizes.push_back(PatchSize{a.n, a.ng});
  return sizes;
}

static RoundCut round_cut(const mgrhd_batch* bt, int64_t chunk) {
  const int threads[2] = {item_threads(false), item_threads(true)};
  return cut_by_rounds(patch_sizes(bt), chunk, device_cus(), threads);
}

static int build_items(mgrhd_batch* bt) {
  CellCut cells = cut_by_cells(patch_sizes(bt), bt->chunk);
  const RoundCut rounds = round_cut(bt, bt->chunk);
  bt->n_items = (int64_t)cells.items.size();
  bt->ng_items.swap(cells.ng_items);
  bt->n_rounds = (int64_t)rounds.items.size();
  bt->n_full = rounds.n_full;
  // (few lanes per cell take room for many cells, many lanes for wide tables)
  bt->lds_rest = bt->lds_full = 0;
  for (int lanes = 1; lanes <= kWave; lanes *= 2) {
    if (rounds.lanes[0] & lanes) bt->lds_rest = std::max(bt->lds_rest, item_lds<false>(lanes));
    if (rounds.lanes[1] & lanes) bt->lds_full = std::max(bt->lds_full, item_lds<true>(lanes));
  }
  if (const int rc = upload_items(cells.items, bt->d_items)) return rc;
  if (const int rc = upload_items(rounds.items, bt->d_rounds)) return rc;
  bt->items_dirty = false;
  return 0;
}

static void drop_graph(mgrhd_batch* bt) {
  if (bt->exec) (void)hipGraphExecDestroy(bt->exec);
  if (bt->graph) (void)hipGraphDestroy(bt->graph);
  bt->exec = nullptr;
  bt->graph = nullptr;
}

extern "C" {

int mgrhd_batch_create(const mgrhd_patch* patches, int32_t n_patches, int32_t mean_mode,
                       const mgrhd_options* opt_in, mgrhd_batch** out) {
  if (!out) return MGRHD_E_NULL;
  *out = nullptr;
  if (n_patches < 0 || (n_patches > 0 && !patches)) return MGRHD_E_NULL;
  if (mean_mode < 0 || mean_mode > 2) return MGRHD_E_MODE;
  mgrhd_options defaults;
  mgrhd_default_options(&defaults);
  const mgrhd_options* opt = opt_in ? opt_in : &defaults;
  if (opt->closure < 0 || opt->closure > 1) return MGRHD_E_MODE;
  if (opt->E_g_out || opt->F_g_out || opt->e_gas_out || opt->v_out)
    return MGRHD_E_OPTION;  // outputs are given per patch
  auto pos = [](double x) { return x > 0.0 && std::isfinite(x); };
  if (!pos(opt->c) || !pos(opt->a_rad) || !pos(opt->h_over_k) || !pos(opt->c_v))
    return MGRHD_E_SCALAR;
  if (!pos(opt->eps_newton) || !pos(opt->eps_outer) || opt->max_newton < 1 ||
      opt->max_outer < 1 || opt->polish < 0 || opt->polish > 4 || opt->guess_kind < 0 ||
      opt->guess_kind > 1)
    return MGRHD_E_OPTION;
  mgrhd_batch* bt = new (std::nothrow) mgrhd_batch();
  if (!bt) return MGRHD_E_DEVICE;
  bt->n_patches = n_patches;
  bt->mode = mean_mode;
  bt->guess_kind = opt->guess_kind;
  bt->h_patches.resize(n_patches);
  for (int32_t p = 0; p < n_patches; ++p) {
    const mgrhd_patch& q = patches[p];
    if (q.n_cells < 0 || q.n_groups < 1 || q.n_groups > kBatchNGM) {
      delete bt;
      return MGRHD_E_SIZE;
    }
    if (q.n_cells > 0 && (!q.E_g || !q.F_g || !q.rho || !q.e_gas || !q.v || !q.group_edges ||
                          !q.chi_lo)) {
      delete bt;
      return MGRHD_E_NULL;
    }
    if (mean_mode != MGRHD_MEAN_PC && !q.alpha_chi && !q.chi_hi) {
      delete bt;
      return MGRHD_E_TABLE;
    }
    if (!pos(q.dt) || !pos(q.c_hat)) {
      delete bt;
      return MGRHD_E_SCALAR;
    }
    const int n_out = !!q.E_g_out + !!q.F_g_out + !!q.e_gas_out + !!q.v_out;
    if (n_out != 0 && n_out != 4) {  // out of place needs all four
      delete bt;
      return MGRHD_E_NULL;
    }
    KArgs& a = bt->h_patches[p];
    std::memset(&a, 0, sizeof(a));
    a.E = q.E_g;
    a.F = q.F_g;
    a.rho = q.rho;
    a.egas = q.e_gas;
    a.v = q.v;
    a.kappa = q.kappa_scale;
    a.S = q.S_g;
    a.guess = q.guess;
    a.guess_kind = opt->guess_kind;
    a.iters = q.iters;
    a.outer = q.outer;
    a.status = q.status;
    a.trace = q.trace;
    a.Eo = q.E_g_out;  // NULL: set_derived points them at the inputs (in place)
    a.Fo = q.F_g_out;
    a.egaso = q.e_gas_out;
    a.vo = q.v_out;
    a.edges = q.group_edges;
    a.chi_lo = q.chi_lo;
    a.alpha = q.alpha_chi;
    a.chi_hi = q.chi_hi;
    a.n = q.n_cells;
    a.ng = q.n_groups;
    a.closure = opt->closure;
    a.dt = q.dt;
    a.chat = q.c_hat;
    a.c = opt->c;
    a.a = opt->a_rad;
    a.hk = opt->h_over_k;
    a.cv = opt->c_v;
    a.eps = opt->eps_newton;
    a.eps_out = opt->eps_outer;
    a.max_newton = opt->max_newton;
    a.max_outer = opt->max_outer;
    a.polish = opt->polish;
    set_derived(a);
    bt->n_cells += q.n_cells;
    bt->max_groups = std::max(bt->max_groups, q.n_groups);
  }
  if (n_patches > 0) {
    if (hipMalloc(&bt->d_patches, sizeof(KArgs) * n_patches) != hipSuccess ||
        hipMemcpy(bt->d_patches, bt->h_patches.data(), sizeof(KArgs) * n_patches,
                  hipMemcpyHostToDevice) != hipSuccess) {
      mgrhd_batch_destroy(bt);
      return MGRHD_E_DEVICE;
    }
  }
  if (hipMalloc(&bt->d_counter, sizeof(int32_t)) != hipSuccess) {
    mgrhd_batch_destroy(bt);
    return MGRHD_E_DEVICE;
  }
  const int rc = build_items(bt);
  if (rc) {
    mgrhd_batch_destroy(bt);
    return rc;
  }
  *out = bt;
  return 0;
}

int mgrhd_batch_set_tuning(mgrhd_batch* bt, int32_t groups_per_lane, int32_t blocks_per_cu,
                           int64_t chunk_cells) {
  if (!bt) return MGRHD_E_NULL;
  if (groups_per_lane != 2 && groups_per_lane != 4) return MGRHD_E_OPTION;
  if (blocks_per_cu < 0 || chunk_cells < 1) return MGRHD_E_OPTION;
  if (bt->max_groups > groups_per_lane * 64) return MGRHD_E_OPTION;
  const bool changed = groups_per_lane != bt->groups_per_lane ||
                       blocks_per_cu != bt->blocks_per_cu || chunk_cells != bt->chunk;
  if (changed) drop_graph(bt);
  bt->groups_per_lane = groups_per_lane;
  bt->blocks_per_cu = blocks_per_cu;
  if (chunk_cells != bt->chunk) {
    // the work lists are rebuilt here, never inside run / capture / launch
    bt->chunk = chunk_cells;
    bt->items_dirty = true;
    return build_items(bt);
  }
  return 0;
}

int mgrhd_batch_set_item_scope(mgrhd_batch* bt, int32_t per_workgroup) {
  if (!bt) return MGRHD_E_NULL;
  if (per_workgroup < 0 || per_workgroup > 2) return MGRHD_E_OPTION;
  if (per_workgroup != bt->scope) {
    bt->scope = per_workgroup;
    drop_graph(bt);
  }
  return 0;
}

int32_t mgrhd_batch_get_item_scope(const mgrhd_batch* bt) {
  return bt ? bt->scope : MGRHD_E_NULL;
}

int mgrhd_batch_get_tuning(const mgrhd_batch* bt, int32_t* groups_per_lane,
                           int32_t* blocks_per_cu, int64_t* chunk_cells) {
  if (!bt) return MGRHD_E_NULL;
  if (groups_per_lane) *groups_per_lane = bt->groups_per_lane;
  if (blocks_per_cu) *blocks_per_cu = bt->blocks_per_cu;
  if (chunk_cells) *chunk_cells = bt->chunk;
  return 0;
}

// the attached networks' inference, one launch per group count
static int enqueue_infer(mgrhd_batch* bt, hipStream_t stream) {
  for (const auto& net : bt->nets)
    for (const auto& r : bt->ng_items)
      if (r.first == net.ng) {
        const int rc = mlp_infer_items(net.m, bt->d_patches, bt->d_items, r.second.first,
                                       r.second.second, net.ng, bt->guess_kind, net.x_mean,
                                       net.x_istd, net.y_mean, net.y_std, stream);
        if (rc) return rc;
      }
  return 0;
}

// One workgroup per item of [lo, hi).  blocks_per_cu caps the workgroups that
// a CU holds at once through the LDS that each asks for.
static int enqueue_items(const mgrhd_batch* bt, hipStream_t stream, bool full, int64_t lo,
                         int64_t hi) {
  if (lo == hi) return 0;
  constexpr size_t kCuLds = 160 * 1024, kLaunchLds = 64 * 1024;
  const ItemsFn fn = items_fn(bt->mode, full);
  size_t lds = full ? bt->lds_full : bt->lds_rest;
  if (bt->blocks_per_cu > 0) {
    const size_t share = kCuLds / (size_t)bt->blocks_per_cu;
    const size_t pad = share / 1024 * 1024;
    if (pad > lds) lds = pad;
  }
  if (lds > kLaunchLds &&
      hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)kCuLds) != hipSuccess)
    return MGRHD_E_DEVICE;
  // a launch holds fewer than 2^32 threads: 8.4e6 items of 512
  const int64_t most = (int64_t)UINT32_MAX / item_threads(full);
  for (; lo < hi; lo += most) {
    hipLaunchKernelGGL(fn, dim3((unsigned)std::min(most, hi - lo)), dim3(item_threads(full)), lds,
                       stream, (const KArgs*)bt->d_patches, (const Item*)(bt->d_rounds + lo));
    if (const hipError_t err = hipGetLastError()) return (int)err;
  }
  return 0;
}

static int enqueue(mgrhd_batch* bt, hipStream_t stream) {
  if (bt->items_dirty) return MGRHD_E_DEVICE;  // the last rebuild of the work list failed
  if (bt->n_items == 0) return 0;
  if (const int rc = enqueue_infer(bt, stream)) return rc;
  if (bt->scope == 1 && bt->groups_per_lane == 2) {
    const int rc = enqueue_items(bt, stream, true, 0, bt->n_full);
    return rc ? rc : enqueue_items(bt, stream, false, bt->n_full, bt->n_rounds);
  }
  BatchFn fn = batch_fn(bt->groups_per_lane, bt->mode, bt->scope);
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, kBlock, 0) != hipSuccess || nb < 1)
    nb = 1;
  if (bt->blocks_per_cu > 0 && bt->blocks_per_cu < nb) nb = bt->blocks_per_cu;
  int64_t blocks = (int64_t)device_cus() * nb;
  // never more takers than items: waves (scope 0) or workgroups (scope 1)
  if (bt->scope) {
    if (blocks > bt->n_items) blocks = bt->n_items;
  } else if (blocks * (kBlock / kWave) > bt->n_items) {
    blocks = (bt->n_items + 3) / 4;
  }
  hipLaunchKernelGGL(k_clear_counter, dim3(1), dim3(64), 0, stream, bt->d_counter);
  BatchArgs args{bt->d_patches, bt->d_items, bt->d_counter, bt->n_items};
  hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(kBlock), 0, stream, args);
  const hipError_t err = hipGetLastError();
  return err == hipSuccess ? 0 : (int)err;
}

int mgrhd_batch_run(mgrhd_batch* bt, mgrhd_stream_t stream) {
  if (!bt) return MGRHD_E_NULL;
  return enqueue(bt, (hipStream_t)stream);
}

int mgrhd_batch_attach_mlp(mgrhd_batch* bt, int32_t n_groups, mgrhd_mlp* m,
                           const float* x_mean, const float* x_istd, const float* y_mean,
                           const float* y_std) {
  if (!bt || !m || !x_mean || !x_istd || !y_mean || !y_std) return MGRHD_E_NULL;
  if (const int rc = mlp_check_patches(m, n_groups)) return rc;
  bool any = false;
  for (const KArgs& a : bt->h_patches)
    if (a.ng == n_groups) {
      if (!a.guess) return MGRHD_E_NULL;  // the inference writes the patch's guess buffer
      any = true;
    }
  if (!any) return MGRHD_E_SIZE;
  for (auto& net : bt->nets)
    if (net.ng == n_groups) {
      net = {n_groups, m, x_mean, x_istd, y_mean, y_std};
      drop_graph(bt);
      return 0;
    }
  bt->nets.push_back({n_groups, m, x_mean, x_istd, y_mean, y_std});
  drop_graph(bt);
  return 0;
}

int mgrhd_batch_infer(mgrhd_batch* bt, mgrhd_stream_t stream) {
  if (!bt) return MGRHD_E_NULL;
  if (bt->items_dirty) return MGRHD_E_DEVICE;
  return enqueue_infer(bt, (hipStream_t)stream);
}

int mgrhd_batch_capture(mgrhd_batch* bt, mgrhd_stream_t stream) {
  if (!bt) return MGRHD_E_NULL;
  drop_graph(bt);
  if (bt->items_dirty) return MGRHD_E_DEVICE;
  hipStream_t st = (hipStream_t)stream;
  hipError_t e = hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) return (int)e;
  const int rc = enqueue(bt, st);
  hipGraph_t g = nullptr;
  e = hipStreamEndCapture(st, &g);
  if (rc) {
    if (g) (void)hipGraphDestroy(g);
    return rc;
  }
  if (e != hipSuccess) return (int)e;
  bt->graph = g;
  e = hipGraphInstantiate(&bt->exec, g, nullptr, nullptr, 0);
  if (e != hipSuccess) {
    drop_graph(bt);
    return (int)e;
  }
  return 0;
}

int mgrhd_batch_launch(mgrhd_batch* bt, mgrhd_stream_t stream) {
  if (!bt) return MGRHD_E_NULL;
  if (!bt->exec) {
    const int rc = mgrhd_batch_capture(bt, stream);
    if (rc) return rc;
  }
  const hipError_t e = hipGraphLaunch(bt->exec, (hipStream_t)stream);
  return e == hipSuccess ? 0 : (int)e;
}

int64_t mgrhd_batch_cells(const mgrhd_batch* bt) { return bt ? bt->n_cells : -1; }

void mgrhd_batch_destroy(mgrhd_batch* bt) {
  if (!bt) return;
  drop_graph(bt);
  if (bt->d_patches) (void)hipFree(bt->d_patches);
  if (bt->d_items) (void)hipFree(bt->d_items);
  if (bt->d_rounds) (void)hipFree(bt->d_rounds);
  if (bt->d_counter) (void)hipFree(bt->d_counter);
  delete bt;
}

// ---------------------------------------------------------------------------
// Autotuner: every candidate launch shape runs on copies of the first
// kTuneCells cells of every patch (restored before each run), timed with HIP
// events; the fastest is kept.  The caller's arrays are only read.
static constexpr int64_t kTuneCells = 1024;

namespace {
struct TuneCandidate {
  int32_t groups_per_lane, scope;
  int64_t chunk;
};
constexpr TuneCandidate kTuneCandidates[] = {
    {2, 0, 1024}, {4, 0, 1024}, {2, 1, 256}, {2, 1, 1024}, {2, 2, 256}, {4, 2, 1024}};

struct TuneBuffers {
  double* pristine = nullptr;
  double* work = nullptr;
  int32_t* ints = nullptr;
  ~TuneBuffers() {
    if (pristine) (void)hipFree(pristine);
    if (work) (void)hipFree(work);
    if (ints) (void)hipFree(ints);
  }
};
}  // namespace

int mgrhd_batch_tune(mgrhd_batch* bt, mgrhd_stream_t stream) {
  if (!bt) return MGRHD_E_NULL;
  if (bt->items_dirty) return MGRHD_E_DEVICE;
  if (bt->n_cells == 0) return 0;
  hipStream_t st = (hipStream_t)stream;
  // sample layout: per patch the first ns cells of every row of every field
  const int32_t np = bt->n_patches;
  std::vector<int64_t> ns(np), off(np);
  int64_t nd = 0, ni = 0;
  auto doubles_of = [&](const KArgs& a, int64_t m) {
    int64_t d = (int64_t)a.ng * m * 4 + m * 5;  // E_g, F_g, rho, e_gas, v
    if (a.kappa) d += m;
    if (a.S) d += (int64_t)a.ng * m;
    if (a.guess) d += a.guess_kind == 1 ? m : (int64_t)(a.ng + 1) * m;
    return d;
  };
  for (int32_t p = 0; p < np; ++p) {
    const KArgs& a = bt->h_patches[p];
    ns[p] = std::min<int64_t>(a.n, kTuneCells);
    off[p] = nd;
    nd += doubles_of(a, ns[p]);
    ni += 3 * ns[p];
  }
  TuneBuffers buf;
  if (hipMalloc(&buf.pristine, sizeof(double) * nd) != hipSuccess ||
      hipMalloc(&buf.work, sizeof(double) * nd) != hipSuccess ||
      hipMalloc(&buf.ints, sizeof(int32_t) * ni) != hipSuccess)
    return MGRHD_E_DEVICE;
  // the sample batch: the same patches over the work copies
  mgrhd_batch tmp;
  tmp.n_patches = np;
  tmp.mode = bt->mode;
  tmp.max_groups = bt->max_groups;
  tmp.h_patches = bt->h_patches;
  int64_t io = 0;
  hipError_t e = hipSuccess;
  for (int32_t p = 0; p < np && e == hipSuccess; ++p) {
    const KArgs& a = bt->h_patches[p];
    KArgs& t = tmp.h_patches[p];
    const int64_t m = ns[p];
    double* w = buf.work + off[p];
    double* q = buf.pristine + off[p];
    // copy `rows` rows of m cells (row pitch a.n) of field src into the sample
    auto take = [&](const double* src, int64_t rows) -> double* {
      if (e == hipSuccess && m > 0)
        e = hipMemcpy2DAsync(q, sizeof(double) * m, src, sizeof(double) * a.n,
                             sizeof(double) * m, rows, hipMemcpyDeviceToDevice, st);
      double* here = w;
      w += rows * m;
      q += rows * m;
      return here;
    };
    t.n = m;
    t.E = take(a.E, a.ng);
    t.F = take(a.F, 3 * (int64_t)a.ng);
    t.rho = take(a.rho, 1);
    t.egas = take(a.egas, 1);
    t.v = take(a.v, 3);
    t.Eo = t.E;  // the trial runs update the copies in place
    t.Fo = t.F;
    t.egaso = t.egas;
    t.vo = t.v;
    t.kappa = a.kappa ? take(a.kappa, 1) : nullptr;
    t.S = a.S ? take(a.S, a.ng) : nullptr;
    t.guess = a.guess ? take(a.guess, a.guess_kind == 1 ? 1 : a.ng + 1) : nullptr;
    t.iters = buf.ints + io;
    t.outer = buf.ints + io + m;
    t.status = buf.ints + io + 2 * m;
    t.trace = nullptr;
    io += 3 * m;
    tmp.n_cells += m;
  }
  if (e != hipSuccess) return MGRHD_E_DEVICE;
  int rc = 0;
  if (hipMalloc(&tmp.d_patches, sizeof(KArgs) * np) != hipSuccess ||
      hipMemcpyAsync(tmp.d_patches, tmp.h_patches.data(), sizeof(KArgs) * np,
                     hipMemcpyHostToDevice, st) != hipSuccess ||
      hipMalloc(&tmp.d_counter, sizeof(int32_t)) != hipSuccess)
    rc = MGRHD_E_DEVICE;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (!rc && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess))
    rc = MGRHD_E_DEVICE;
  float best_ms = 0.f;
  const TuneCandidate* best = nullptr;
  int64_t best_chunk = 0;
  // the work lists of the candidates of one workgroup per item so far: there the
  // cells per item are a cap that a sample may never reach, and a list that was
  // timed is not timed again
  std::vector<RoundCut> timed;
  for (const TuneCandidate& c : kTuneCandidates) {
    if (rc) break;
    if (bt->max_groups > c.groups_per_lane * 64) continue;
    int64_t chunk = c.chunk;
    if (c.scope == 1 && c.groups_per_lane == 2) {
      RoundCut cut = round_cut(&tmp, c.chunk);
      bool seen = false;
      for (const RoundCut& t : timed) seen = seen || t.items == cut.items;
      if (seen) continue;
      // nor does such a sample tell this cap from the batch's own, which then stays
      if (round_cut(&tmp, bt->chunk).items == cut.items) chunk = bt->chunk;
      timed.push_back(std::move(cut));
    }
    tmp.groups_per_lane = c.groups_per_lane;
    tmp.scope = c.scope;
    tmp.blocks_per_cu = bt->blocks_per_cu;
    if (c.chunk != tmp.chunk || tmp.items_dirty) {
      tmp.chunk = c.chunk;
      if (hipStreamSynchronize(st) != hipSuccess) { rc = MGRHD_E_DEVICE; break; }
      if ((rc = build_items(&tmp)) != 0) break;
    }
    float ms = 0.f;
    for (int rep = 0; rep < 2 && !rc; ++rep) {  // the first run warms up
      if (hipMemcpyAsync(buf.work, buf.pristine, sizeof(double) * nd, hipMemcpyDeviceToDevice,
                         st) != hipSuccess ||
          hipEventRecord(e0, st) != hipSuccess)
        rc = MGRHD_E_DEVICE;
      if (!rc) rc = enqueue(&tmp, st);
      if (!rc && (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                  hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
        rc = MGRHD_E_DEVICE;
    }
    if (!rc && (!best || ms < best_ms)) {
      best = &c;
      best_ms = ms;
      best_chunk = chunk;
    }
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipStreamSynchronize(st);
  if (tmp.d_patches) (void)hipFree(tmp.d_patches);
  if (tmp.d_items) (void)hipFree(tmp.d_items);
  if (tmp.d_rounds) (void)hipFree(tmp.d_rounds);
  if (tmp.d_counter) (void)hipFree(tmp.d_counter);
  if (rc) return rc;
  if (!best) return MGRHD_E_OPTION;
  rc = mgrhd_batch_set_tuning(bt, best->groups_per_lane, bt->blocks_per_cu, best_chunk);
  if (!rc) rc = mgrhd_batch_set_item_scope(bt, best->scope);
  return rc;
}

}  // extern "C"
