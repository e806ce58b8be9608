"""CPU test of the split length of a selected-token plan: the header the kernel uses, compiled for the host."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_16928_amd", "csrc")


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    assert cxx, "a host C++ compiler is needed"
    d = tmp_path_factory.mktemp("split")
    (d / "split.cpp").write_text('#include "split_plan.h"\nextern "C" int split(int t, int l, int n) { return rtp::split_blocks(t, l, n); }\n')
    so = str(d / "split.so")
    subprocess.run([cxx, "-std=c++17", "-O2", "-shared", "-fPIC", "-w", "-D__host__=", "-D__device__=", "-D__forceinline__=inline",
                    "-I", CSRC, str(d / "split.cpp"), "-o", so], check=True)
    return C.CDLL(so).split


@pytest.mark.parametrize("units,long_units", [(1, 1), (2, 1), (2, 2), (12, 1), (64, 1), (64, 64), (1024, 3), (1024, 1024)])
@pytest.mark.parametrize("tokens", [1, 128, 129, 8192, 8193, 16384, 32768, 40000, 65536, 131072, 1 << 20])
def test_items_of_a_plan(split, units, long_units, tokens):
    """Few partials for the one workgroup that merges a unit unless its items have their full length, an item for each of 256
    compute units where there are enough blocks for that, and never more items than the workspace holds partials."""
    blocks = [-(-tokens // 128)] * long_units + [1] * (units - long_units)
    total, longest = sum(blocks), max(blocks)
    target = min(1024, units * longest)                    # the host's: the bound of every unit is the longest one's
    st = split(total, longest, target)
    items = sum(-(-b // st) for b in blocks)
    assert st >= 1 and items <= target + units
    assert -(-longest // st) <= 64 or st >= 5
    assert st <= 5 or st == -(-total // target)
    if st > 1 and -(-longest // (st - 1)) <= 64 and st <= 5:
        assert sum(-(-b // (st - 1)) for b in blocks) >= 256


def test_an_empty_plan(split):
    assert split(0, 0, 0) == 1 and split(0, 0, 1024) == 1
