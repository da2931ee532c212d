// Host build of the batch's work lists, for the CPU test suite.
#include "../../paper_2407_18304_amd/csrc/batch_items.hpp"

using namespace mgrhd;

static std::vector<PatchSize> sizes(const int64_t* n, const int32_t* ng, int32_t patches) {
  std::vector<PatchSize> s;
  for (int32_t p = 0; p < patches; ++p) s.push_back(PatchSize{n[p], ng[p]});
  return s;
}
static int64_t give(const std::vector<BatchItem>& items, int64_t* out, int64_t room) {
  for (int64_t k = 0; k < (int64_t)items.size() && k < room; ++k) {
    out[3 * k] = items[k].patch;
    out[3 * k + 1] = items[k].c0;
    out[3 * k + 2] = items[k].c1;
  }
  return (int64_t)items.size();
}

extern "C" {
// (patch, c0, c1) of the first `room` items; returns the number of all
int64_t bi_cells(const int64_t* n, const int32_t* ng, int32_t patches, int64_t chunk, int64_t* out,
                 int64_t room) {
  return give(cut_by_cells(sizes(n, ng, patches), chunk).items, out, room);
}
int64_t bi_rounds(const int64_t* n, const int32_t* ng, int32_t patches, int64_t chunk, int64_t cus,
                  int32_t rest, int32_t full, int64_t* out, int64_t room, int64_t* n_full,
                  int32_t* lanes) {
  const int threads[2] = {rest, full};
  const RoundCut c = cut_by_rounds(sizes(n, ng, patches), chunk, cus, threads);
  *n_full = c.n_full;
  lanes[0] = c.lanes[0];
  lanes[1] = c.lanes[1];
  return give(c.items, out, room);
}
}
