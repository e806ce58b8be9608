// The scan of a prefill threshold search's histogram (attn_prefill.hip), apart from the kernel so that host code can run it too.
#pragma once

namespace rtp {

struct ThresholdBin {
  int bin;             // where the descending cumulative mass reaches the target
  double above, mass;  // mass above that bin, and its own
};

// `above` is the mass above bin 0, rs[] the sums of RUNS runs of RUN_BINS bins each, mass_of(i) the mass of bin i.  The run is found
// from the sums, the bin from the run's bins one by one.  The two add up in different orders, so a target within a rounding error
// of the run's end can be reached by the run and by none of its bins: then it is the last bin of the run that holds any mass.
template <int RUNS, int RUN_BINS, class MassOf>
__host__ __device__ __forceinline__ ThresholdBin threshold_bin(const double above, const double target, const double (&rs)[RUNS],
                                                               const MassOf& mass_of) {
  double cum = above;
  int run = RUNS - 1;
  bool found = false;
#pragma unroll
  for (int i = 0; i < RUNS - 1; ++i) {
    found = found || cum + rs[i] >= target;
    if (!found) cum += rs[i];
    else run = run < i ? run : i;
  }
  ThresholdBin t = {RUNS * RUN_BINS - 1, 0.0, 0.0};
  found = false;
  const double before_run = cum;
  double h[RUN_BINS];
#pragma unroll
  for (int i = 0; i < RUN_BINS; ++i) h[i] = mass_of(run * RUN_BINS + i);
#pragma unroll
  for (int i = 0; i < RUN_BINS; ++i) {
    if (!found) {
      if (cum + h[i] >= target) { t.bin = run * RUN_BINS + i; t.mass = h[i]; found = true; }
      else cum += h[i];
    }
  }
  t.above = cum;
  if (!found) {          // (hardly ever: a branch of its own keeps it out of the walk)
    cum = before_run;
#pragma unroll
    for (int i = 0; i < RUN_BINS; ++i) {
      if (h[i] > 0.0) t = {run * RUN_BINS + i, cum, h[i]};
      cum += h[i];
    }
  }
  return t;
}

}  // namespace rtp
