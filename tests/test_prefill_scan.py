"""CPU test of the histogram scan of the prefill threshold search: the header the kernel uses, compiled for the host."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_16928_amd", "csrc")
RUNS, RUN_BINS = 16, 8
BINS = RUNS * RUN_BINS

SOURCE = """
#include "prefill_scan.h"
extern "C" int scan(double above, double target, const double* h, double* above_out, double* mass) {
  double rs[%d];
  for (int k = 0; k < %d; ++k) {
    rs[k] = 0.0;
    for (int i = 0; i < %d; ++i) rs[k] += h[k * %d + i];
  }
  const rtp::ThresholdBin t = rtp::threshold_bin<%d, %d>(above, target, rs, [&](int i) { return h[i]; });
  *above_out = t.above;
  *mass = t.mass;
  return t.bin;
}
// h: n slices of running sums per run
extern "C" int scan_slices(int n, double above, double target, const double* h, double* above_out, double* mass) {
  auto over = [&](int bin) { double s = 0.0; for (int k = 0; k < n; ++k) s += h[k * %d + bin]; return s; };
  double rs[%d], c[%d];
  for (int k = 0; k < %d; ++k) rs[k] = over(k * %d + %d - 1);
  const rtp::ThresholdRun run = rtp::threshold_run<%d>(above, target, rs);
  for (int i = 0; i < %d; ++i) c[i] = over(run.run * %d + i);
  const rtp::ThresholdBin t = rtp::threshold_in_run<%d, %d>(run, target, c);
  *above_out = t.above;
  *mass = t.mass;
  return t.bin;
}
""" % (RUNS, RUNS, RUN_BINS, RUN_BINS, RUNS, RUN_BINS, RUNS * RUN_BINS, RUNS, RUN_BINS, RUNS, RUN_BINS, RUN_BINS, RUNS, RUN_BINS,
       RUN_BINS, RUNS, RUN_BINS)


@pytest.fixture(scope="module")
def scan(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    assert cxx, "a host C++ compiler is needed"
    d = tmp_path_factory.mktemp("scan")
    (d / "scan.cpp").write_text(SOURCE)
    so = str(d / "scan.so")
    subprocess.run([cxx, "-std=c++17", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-w", "-D__host__=", "-D__device__=",
                    "-D__forceinline__=inline", "-I", CSRC, str(d / "scan.cpp"), "-o", so], check=True)
    lib = C.CDLL(so)
    dp = C.POINTER(C.c_double)
    lib.scan.argtypes = [C.c_double, C.c_double, dp, dp, dp]

    def call(above, target, h):
        a, m = C.c_double(), C.c_double()
        b = lib.scan(above, target, h.ctypes.data_as(dp), C.byref(a), C.byref(m))
        return b, a.value, m.value
    call.lib = lib
    return call


def _check(h, above, target, got, what):
    """The bin reaches the target, and the bins before it do not, up to the rounding of 129 additions of the total."""
    b, ab, m = got
    before = above + np.concatenate([[0.0], np.cumsum(h.astype(np.longdouble))]).astype(np.longdouble)
    tol = 129 * 2.0 ** -53 * float(before[-1])
    assert before[b + 1] >= target - tol and before[b] <= target + tol, (what, b, float(before[b]), target)
    assert m == h[b] and abs(ab - float(before[b])) <= tol, (what, b)
    assert m > 0, (what, b)


@pytest.mark.parametrize("empty", [0.0, 0.5, 0.9])
@pytest.mark.parametrize("above", [0.0, 137.25])
def test_scan_with_targets_on_the_ends_of_runs(scan, empty, above):
    """Targets that the running sum over a run reaches exactly, while the bins added one by one may fall short by a rounding."""
    rng = np.random.default_rng(11)
    for k in range(2000):
        h = np.exp(rng.uniform(-12, 6, BINS)) * rng.uniform(0.5, 1.5, BINS)
        h[rng.random(BINS) < empty] = 0.0
        if h.max() == 0.0:
            continue
        cum, ends = above, []
        for run in range(RUNS):
            s = 0.0
            for v in h[run * RUN_BINS:(run + 1) * RUN_BINS]:
                s += v
            cum += s
            if s > 0.0:
                ends.append(cum)
        target = ends[rng.integers(len(ends))]
        _check(h, above, target, scan(above, target, h), (empty, above, k))


def test_scan_with_targets_anywhere(scan):
    rng = np.random.default_rng(12)
    for k in range(2000):
        h = np.exp(rng.uniform(-12, 6, BINS))
        h[rng.random(BINS) < rng.choice([0.0, 0.5, 0.97])] = 0.0
        if h.max() == 0.0:
            continue
        target = float(np.float32(rng.uniform(1e-4, 0.999999))) * float(h.sum())
        _check(h, 0.0, target, scan(0.0, target, h), k)


@pytest.mark.parametrize("n", [2, 3, 16])
@pytest.mark.parametrize("above", [0.0, 41.5])
def test_scan_of_running_sums_in_slices(scan, n, above):
    """What the slices of a search leave (running sums per run) against the masses themselves: targets on the ends of runs as they
    add up there, and anywhere; empty bins in some slices or in all."""
    lib = scan.lib
    dp = C.POINTER(C.c_double)
    lib.scan_slices.argtypes = [C.c_int, C.c_double, C.c_double, dp, dp, dp]
    rng = np.random.default_rng(13 + n)
    for k in range(1500):
        h = np.exp(rng.uniform(-12, 6, (n, BINS))) * rng.uniform(0.5, 1.5, (n, BINS))
        h[rng.random((n, BINS)) < rng.choice([0.0, 0.5, 0.97])] = 0.0
        h[:, rng.random(BINS) < rng.choice([0.0, 0.9])] = 0.0
        if h.max() == 0.0:
            continue
        c = np.ascontiguousarray(np.cumsum(h.reshape(n, RUNS, RUN_BINS), axis=2).reshape(n, BINS))
        whole = c[0].copy()
        for i in range(1, n):
            whole += c[i]
        cum, ends = above, []
        for s in whole[RUN_BINS - 1::RUN_BINS]:
            cum += s
            if s > 0.0:
                ends.append(cum)
        target = ends[rng.integers(len(ends))] if k % 2 else above + float(rng.uniform(1e-4, 0.999999)) * float(h.sum())
        a, m = C.c_double(), C.c_double()
        b = lib.scan_slices(n, above, target, c.ctypes.data_as(dp), C.byref(a), C.byref(m))
        before = above + np.concatenate([[0.0], np.cumsum(h.sum(axis=0, dtype=np.longdouble))]).astype(np.longdouble)
        tol = (129 + n) * 2.0 ** -53 * float(before[-1])                # one rounding per addition, each below the total
        assert before[b + 1] >= target - tol and before[b] <= target + tol, (k, b)
        assert m.value > 0 and abs(m.value - float(h[:, b].sum())) <= tol and abs(a.value - float(before[b])) <= tol, (k, b)
