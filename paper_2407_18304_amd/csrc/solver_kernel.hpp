// solver_kernel.hpp -- the single-table source-update kernel and the list of
// its compiled variants, shared by the four translation units that
// instantiate it (T-independent or T-dependent opacity, any N_g or
// N_g = LPC * G: source_update.hip, source_update_tdep.hip,
// source_update_full.hip, source_update_tdep_full.hip, compiled in parallel).
#pragma once
#include <hip/hip_runtime.h>

#include "solver_device.hpp"

namespace mgrhd {

// LDS of one workgroup of the state machine with LPC lanes per cell: the group
// tables, the per-lane slots, the per-cell area, and the cells of the
// workgroup's range handed out so far.  AT_USE: LaneStore's CONST_AT_USE.
template <int G, int LPC, int THREADS, bool AT_USE = false>
struct BlockLds {
  static constexpr int kThreads = THREADS;
  using LS = LaneStore<G, true, kThreads / LPC, AT_USE, kThreads>;
  Tables<G * LPC> tab;
  double lane[LS::kSlots * kThreads];
  double cell[LS::kCellWords];
  int taken;
};

// The cells [lo, hi) of one state by this workgroup: its tables staged, the
// cells shared by its waves through the counter in LDS.  ap: the argument
// block that a was read from.
template <int G, int LPC, int MODE, bool TD, bool FULL, int THREADS, bool AT_USE>
__device__ __forceinline__ void run_block(const KArgs& a, KArgsRef ap, int64_t lo, int64_t hi,
                                          BlockLds<G, LPC, THREADS, AT_USE>& lds) {
  constexpr int NGM = G * LPC;
  using LS = typename BlockLds<G, LPC, THREADS, AT_USE>::LS;
  const LS ls{lds.lane + threadIdx.x, lds.cell, ap};
  if (threadIdx.x == 0) lds.taken = 0;
  const bool table_ok = stage_tables<NGM, MODE>(a, lds.tab);  // (its barriers publish `taken`)

  if (!table_ok) {
    // the table is unusable: report every cell of this workgroup's range
    for (int64_t i = lo + threadIdx.x; i < hi; i += blockDim.x) {
      copy_through(a, state_ptrs(ap), i, 0, 1);
      if (a.status) a.status[i] = MGRHD_ST_BAD_TABLE;
      if (a.iters) a.iters[i] = 0;
      if (a.outer) a.outer[i] = 0;
      if (a.trace)
        for (int k = 0; k < a.max_outer; ++k) a.trace[(int64_t)k * a.n + i] = -1;
    }
    return;
  }

  run_cells<G, LPC, MODE, NGM, TD, FULL>(a, lds.tab, ls, threadIdx.x % kWave,
                                         BlockQueue{&lds.taken, lo, hi});
}

// TD: the opacity depends on temperature (evaluated at every iterate).
// FULL: N_g = LPC * G (the launcher checks), every slot holds a group.
// Without the per-slot checks the FULL kernels of two groups per lane fit the
// 128 registers of four waves per SIMD, whatever the variant asks for (2^21
// cells x 16 groups 4.35 -> 4.00 ms, PPL-free 5% faster; with the checks they
// would spill: 11 groups 1.19 -> 1.47 ms).  PPL-free with a temperature-dependent
// opacity does not: at four waves it spills, and at 64 groups the compiler then
// puts copies of split registers before the end of a branch's lanes, so that the
// other lanes go on with stale ones.  It keeps three waves.
template <int G, int MODE, int WPE, bool TD, bool FULL>
constexpr int waves_per_simd() {
  if (four_waves<G, FULL, MODE, TD>()) return WPE < 4 ? 4 : WPE;
  return FULL && G == 2 && WPE > 3 ? 3 : WPE;
}
template <int G, int LPC, int MODE, int WPE, bool TD, bool FULL>
__global__ __launch_bounds__((block_threads<G, FULL, MODE, TD>()), WPE) void
k_source_update(KArgs a) {
  __shared__ BlockLds<G, LPC, block_threads<G, FULL, MODE, TD>()> lds;
  // the arguments as the device reads them in place (a is the only argument)
  const KArgsRef ap = (KArgsRef)__builtin_amdgcn_kernarg_segment_ptr();
  // each workgroup owns a contiguous range of cells, shared by its waves
  int64_t lo, hi;
  block_range(a, blockIdx.x, lo, hi);
  run_block<G, LPC, MODE, TD, FULL>(a, ap, lo, hi, lds);
}

using KernelFn = void (*)(KArgs);

// The kernel of a variant: variants that differ only in a budget that
// waves_per_simd sets anyway share one.
template <int G, int LPC, int MODE, int WPE, bool TD, bool FULL>
constexpr KernelFn variant_kernel() {
  return k_source_update<G, LPC, MODE, waves_per_simd<G, MODE, WPE, TD, FULL>(), TD, FULL>;
}

// (groups per lane, lanes per cell, minimum waves per SIMD) of every compiled
// variant.  The first entry of each (lanes per cell, groups per lane) pair is
// its default register budget; the others trade registers (spills) for waves.
#define MGRHD_FOR_EACH_VARIANT(X)                                                 \
  X(4, 1, 2) X(4, 2, 2) X(4, 4, 2) X(4, 8, 2) X(4, 16, 2) X(4, 32, 2) X(4, 64, 2) \
  X(2, 2, 3) X(2, 4, 3) X(2, 8, 3) X(2, 16, 3) X(2, 32, 3)                        \
  X(1, 4, 4) X(1, 8, 4) X(1, 16, 4) X(1, 32, 4) X(1, 64, 4)                       \
  X(2, 8, 4) X(2, 32, 4)

// the three mean modes of one variant
#define MGRHD_VARIANT_MODES(G_, LPC_, WPE_, TD_, FULL_)                            \
  {                                                                               \
    variant_kernel<G_, LPC_, MGRHD_MEAN_PC, WPE_, TD_, FULL_>(),                  \
        variant_kernel<G_, LPC_, MGRHD_MEAN_PPL_FIXED, WPE_, TD_, FULL_>(),       \
        variant_kernel<G_, LPC_, MGRHD_MEAN_PPL_FREE, WPE_, TD_, FULL_>()         \
  }

// A kernel table: the kernel of variant k (in MGRHD_FOR_EACH_VARIANT order)
// and mean mode, or nullptr; the including file defines MGRHD_TABLE_ROW.
#define MGRHD_DEFINE_KERNEL_TABLE(NAME)                                            \
  KernelFn NAME(int k, int mode) {                                                \
    static const KernelFn fns[][3] = {MGRHD_FOR_EACH_VARIANT(MGRHD_TABLE_ROW)};   \
    constexpr int n = (int)(sizeof(fns) / sizeof(fns[0]));                        \
    if (k < 0 || k >= n || mode < 0 || mode > 2) return nullptr;                  \
    return fns[k][mode];                                                          \
  }

// The kernels of the other three translation units, by variant and mode.
KernelFn tdep_kernel(int k, int mode);       // TD, any N_g (source_update_tdep.hip)
KernelFn full_kernel(int k, int mode);       // N_g = LPC * G (source_update_full.hip)
KernelFn tdep_full_kernel(int k, int mode);  // both (source_update_tdep_full.hip)

}  // namespace mgrhd
