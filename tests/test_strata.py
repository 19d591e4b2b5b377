"""The FP32 sum of a pass (csrc/strata.h, compiled here by the host compiler):
the error bound counts every term that a lane adds, and a stratum per lane is
chosen only where half of the lanes have one."""

import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#include "strata.h"
extern "C" int by_lane(unsigned rx, unsigned zc, unsigned lanes) { return bns::strata_by_lane(rx, zc, lanes); }
extern "C" double terms(unsigned rxy, unsigned zc, unsigned lanes, int by) { return bns::lane_terms(rxy, zc, lanes, by != 0); }
extern "C" double bound(double terms, unsigned passes) { return bns::fp32_sum_bound(terms, passes); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("strata")
    (d / "strata.cpp").write_text(SRC)
    so = d / "strata.so"
    subprocess.run([gxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-D__host__=", "-D__device__=", "-I",
                    os.path.join(ROOT, "paper_2212_04259_amd", "csrc"), str(d / "strata.cpp"), "-o", str(so)],
                   check=True, capture_output=True)
    L = ctypes.CDLL(str(so))
    L.bound.restype = ctypes.c_double
    L.bound.argtypes = [ctypes.c_double, ctypes.c_uint]
    L.terms.restype = ctypes.c_double
    return L


@pytest.mark.parametrize("lanes,words", [(64, 1600), (256, 6400), (256, 10240)])
@pytest.mark.parametrize("rx", [2, 3, 4, 5, 6, 9])
@pytest.mark.parametrize("ry", [2, 3, 5, 15, 60, 200])
def test_terms_and_lanes(lib, lanes, words, rx, ry):
    rxy = rx * ry
    full = (words - lanes) // (rxy + rx + ry + 1)  # strata of a full pass
    for zc in sorted({1, max(1, full // 3), full} - {0}):
        by = lib.by_lane(rx, zc, lanes)
        if by:
            assert 2 <= rx <= 5 and min(zc, lanes) >= lanes / 2
            per_lane = [rxy * len(range(r, zc, lanes)) for r in range(lanes)]
        else:
            per_lane = [len(range(r, rxy * zc, lanes)) for r in range(lanes)]
        most = lib.terms(rxy, zc, lanes, by)
        assert max(per_lane) <= most
        if not by:  # as for every sum by cells (batches of tests, one-pass tables)
            assert most == rxy * zc / lanes + 1
        # a sum of k terms in FP32, each with 32 ulp of its own, then a tree of the lanes
        assert lib.bound(most, 3) >= 3 * (32 + max(per_lane)) * 2.0 ** -24
