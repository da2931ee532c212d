// batch_items.hpp -- how the patches of a batch are cut into work items (host
// code only).  A batch keeps two lists of the same cells: one cut by cells, for
// the kernels that take items from a counter and for the network's inference,
// and one cut by rounds, for the launch of one workgroup per item.
#pragma once
#include <algorithm>
#include <cstdint>
#include <utility>
#include <vector>

namespace mgrhd {

// cells [c0, c1) of patch `patch`
struct BatchItem {
  int32_t patch;
  int32_t pad;
  int64_t c0, c1;
};
inline bool operator==(const BatchItem& a, const BatchItem& b) {
  return a.patch == b.patch && a.c0 == b.c0 && a.c1 == b.c1;
}

struct PatchSize {
  int64_t n;
  int32_t ng;
};

// Lanes per cell of N_g groups at 2 groups per lane, and whether the groups
// fill them.
inline int item_lanes(int ng) {
  int lanes = 1;
  while (lanes * 2 < ng) lanes <<= 1;
  return lanes;
}
inline bool fills_lanes(int ng) { return 2 * item_lanes(ng) == ng; }

// Items of at most `chunk` cells, by decreasing N_g (the costliest first), and
// the [first, last) item of each group count.
struct CellCut {
  std::vector<BatchItem> items;
  std::vector<std::pair<int32_t, std::pair<int64_t, int64_t>>> ng_items;
};
inline CellCut cut_by_cells(const std::vector<PatchSize>& patches, int64_t chunk) {
  std::vector<int32_t> order(patches.size());
  for (size_t p = 0; p < order.size(); ++p) order[p] = (int32_t)p;
  std::stable_sort(order.begin(), order.end(),
                   [&](int32_t x, int32_t y) { return patches[x].ng > patches[y].ng; });
  CellCut cut;
  for (int32_t p : order) {
    const int64_t n = patches[p].n, at = (int64_t)cut.items.size();
    if (cut.ng_items.empty() || cut.ng_items.back().first != patches[p].ng)
      cut.ng_items.push_back({patches[p].ng, {at, at}});
    for (int64_t c0 = 0, c1; c0 < n; c0 = c1) {
      c1 = n - c0 > chunk ? c0 + chunk : n;
      cut.items.push_back(BatchItem{p, 0, c0, c1});
    }
    cut.ng_items.back().second.second = (int64_t)cut.items.size();
  }
  return cut;
}

// Items for one workgroup each (k_batch_items): those of patches whose groups
// fill their lanes first (a launch of its own), each part by decreasing N_g.
// The length of an item counts in rounds of the cells that a workgroup holds
// at once, not in cells: as many rounds for a narrow patch as for a wide one,
// and, as the hardware starts item after item, half of what the launch has left
// for each resident workgroup, so that all end together (block_range).
// Measured: 24 patches of 1.3e6 cells 8.29 ms with 256 cells per item, 2.4 ms of
// it the last items of 64 groups.  `chunk` caps an item of 32 lanes per cell,
// and one of fewer lanes at as many times more cells as run side by side.
struct RoundCut {
  std::vector<BatchItem> items;
  int64_t n_full = 0;       // the first items, of patches that fill their lanes
  int lanes[2] = {0, 0};    // lanes per cell (powers of two) that occur, ORed: others, full
};
inline RoundCut cut_by_rounds(const std::vector<PatchSize>& patches, int64_t chunk, int64_t cus,
                              const int (&threads)[2]) {
  constexpr int64_t kLeastRounds = 2;
  std::vector<int32_t> order(patches.size());
  for (size_t p = 0; p < order.size(); ++p) order[p] = (int32_t)p;
  auto full = [&](int32_t p) { return fills_lanes(patches[p].ng); };
  std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
    if (full(x) != full(y)) return full(x);
    return patches[x].ng > patches[y].ng;
  });
  auto in_flight = [&](int32_t p) {
    return (int64_t)(threads[full(p)] / item_lanes(patches[p].ng));
  };
  int64_t left[2] = {0, 0};  // rounds left of the others and of the full items
  for (int32_t p : order) left[full(p)] += (patches[p].n + in_flight(p) - 1) / in_flight(p);
  // workgroups on the chip: three waves per SIMD of the others, four of the full items
  const int64_t on_chip[2] = {cus * 12 * 64 / threads[0], cus * 16 * 64 / threads[1]};
  RoundCut cut;
  for (int32_t p : order) {
    const int64_t n = patches[p].n, held = in_flight(p);
    const int lanes = item_lanes(patches[p].ng), f = full(p);
    // chunk * 32 / lanes, at least a cell, without overflow
    const int64_t more = lanes < 32 ? 32 / lanes : 1, fewer = lanes > 32 ? lanes / 32 : 1;
    const int64_t most =
        chunk > INT64_MAX / more ? INT64_MAX : std::max<int64_t>(chunk * more / fewer, 1);
    for (int64_t c0 = 0, c1; c0 < n; c0 = c1) {
      const int64_t r = std::max(left[f] / (2 * on_chip[f]), kLeastRounds);
      const int64_t cells = std::min(std::min(r * held, most), n - c0);
      left[f] -= (cells + held - 1) / held;
      c1 = c0 + cells;
      cut.items.push_back(BatchItem{p, 0, c0, c1});
    }
    if (n > 0) cut.lanes[f] |= lanes;
    if (f) cut.n_full = (int64_t)cut.items.size();
  }
  return cut;
}

}  // namespace mgrhd
