// The scan of a prefill threshold search's histogram (attn_prefill.hip), apart from the kernel so that host code can run it too.
#pragma once

namespace rtp {

struct ThresholdBin {
  int bin;             // where the descending cumulative mass reaches the target
  double above, mass;  // mass above that bin, and its own
};

struct ThresholdRun {
  int run;             // the run of bins that reaches the target (the last one if none does)
  double above;        // mass above it
};
template <int RUNS>
__host__ __device__ __forceinline__ ThresholdRun threshold_run(const double above, const double target, const double (&rs)[RUNS]) {
  ThresholdRun t = {RUNS - 1, above};
  bool found = false;
#pragma unroll
  for (int i = 0; i < RUNS - 1; ++i) {
    found = found || t.above + rs[i] >= target;
    if (!found) t.above += rs[i];
    else t.run = t.run < i ? t.run : i;
  }
  return t;
}

// The bin of a run given by its running sums c[], the last of which is the run's sum: a run found by that sum always has a bin
// that reaches the target.  Where the target lies beyond the last run
// as well, the last bin of it that holds any mass.
template <int RUNS, int RUN_BINS>
__host__ __device__ __forceinline__ ThresholdBin threshold_in_run(const ThresholdRun run, const double target, const double (&c)[RUN_BINS]) {
  ThresholdBin t = {RUNS * RUN_BINS - 1, run.above + c[RUN_BINS - 1], 0.0};
  bool found = false;
  double prev = 0.0;
#pragma unroll
  for (int i = 0; i < RUN_BINS; ++i) {
    if (!found && c[i] > prev) t = {run.run * RUN_BINS + i, run.above + prev, c[i] - prev};
    found = found || run.above + c[i] >= target;
    prev = c[i];
  }
  return t;
}

// `above` is the mass above bin 0, rs[] the sums of RUNS runs of RUN_BINS bins each, mass_of(i) the mass of bin i.  The run is found
// from the sums, the bin from the run's bins one by one.  The two add up in different orders, so a target within a rounding error
// of the run's end can be reached by the run and by none of its bins: then it is the last bin of the run that holds any mass.
template <int RUNS, int RUN_BINS, class MassOf>
__host__ __device__ __forceinline__ ThresholdBin threshold_bin(const double above, const double target, const double (&rs)[RUNS],
                                                               const MassOf& mass_of) {
  const ThresholdRun tr = threshold_run<RUNS>(above, target, rs);
  const int run = tr.run;
  double cum = tr.above;
  ThresholdBin t = {RUNS * RUN_BINS - 1, 0.0, 0.0};
  bool found = false;
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
