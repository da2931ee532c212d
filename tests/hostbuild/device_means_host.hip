// Host build of the group-mean inner functions of the source-update kernels,
// for the CPU test suite.  Test infrastructure.
#include "../../paper_2407_18304_amd/csrc/planck_device.hpp"

extern "C" {
void dm_one_minus_exp(double t, double* out) {
  const mgrhd::OneMinusExp o = mgrhd::one_minus_exp(t);
  out[0] = o.em;
  out[1] = o.e;
}
double dm_log_pos(double x) { return mgrhd::log_pos(x); }
double dm_mean_ratio_rac(double ac, double aq, double L, double rac) {
  return mgrhd::mean_ratio_rac(ac, aq, L, rac);
}
double dm_mean_fixed_rac(double y, double rac) { return mgrhd::mean_fixed_rac(y, rac); }
}
