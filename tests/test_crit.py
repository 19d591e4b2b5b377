"""Critical values of the chi-square distribution (csrc/crit.h, compiled here by
the host compiler) against scipy, and the degrees of freedom they are made
for.  The header states quantiles to a part in 10^5."""

import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest
from scipy.stats import chi2

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CRIT_DF = 96
SRC = """
#include "crit.h"
using namespace bns;
extern "C" double half_quantile(int df, double q) { return chi2_half_quantile(df, q, normal_upper(q)).x; }
extern "C" int values(double alpha, double band, int fp64, const unsigned char *need, double *out) {
    CritMask m{};
    for (int d = 0; d < kCritDf; ++d) m[(size_t)d] = need[d] != 0;
    crit_values(alpha, band, fp64 != 0, m, (CritVal *)out);
    return (int)(sizeof(CritVal) / sizeof(double));
}
extern "C" void needed(const unsigned char *card, int top, int adjusted, unsigned char *out) {
    bool c[16] = {};
    for (int a = 0; a <= top; ++a) c[a] = card[a] != 0;
    const CritMask m = crit_need(c, top, adjusted != 0);
    for (int d = 0; d < kCritDf; ++d) out[d] = m[(size_t)d];
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("crit")
    (d / "crit.cpp").write_text(SRC)
    so = d / "crit.so"
    subprocess.run([gxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2212_04259_amd", "csrc"), str(d / "crit.cpp"), "-o", str(so)],
                   check=True, capture_output=True)
    L = ctypes.CDLL(str(so))
    L.half_quantile.restype = ctypes.c_double
    L.half_quantile.argtypes = [ctypes.c_int, ctypes.c_double]
    L.values.argtypes = [ctypes.c_double, ctypes.c_double, ctypes.c_int, ctypes.c_char_p, ctypes.c_void_p]
    L.needed.argtypes = [ctypes.c_char_p, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    return L


def _values(L, alpha, band, need, fp64=0):
    out = np.zeros(8 * CRIT_DF)
    k = L.values(alpha, band, fp64, bytes(bytearray(need)), out.ctypes.data)
    return out[:k * CRIT_DF].reshape(CRIT_DF, k)


@pytest.mark.parametrize("q", [1e-90, 1e-30, 1e-9, 1e-4, 1e-3, 0.01, 0.05, 0.3, 0.5, 0.8, 0.99, 1 - 1e-6, 1 - 1e-9])
def test_quantiles(lib, q):
    for df in range(1, CRIT_DF):
        x = 2.0 * lib.half_quantile(df, q)
        lo, hi = chi2.logsf(x * (1 + 1e-5), df), chi2.logsf(x * (1 - 1e-5), df)
        assert lo <= np.log(q) <= hi, (df, q, x)


@pytest.mark.parametrize("alpha", [1e-20, 1e-6, 1e-4, 0.001, 0.01, 0.05, 0.5, 0.9, 0.9995])
@pytest.mark.parametrize("band", [0.0, 1e-3, 0.2])
def test_values_enclose_the_band(lib, alpha, band):
    need = [1] * CRIT_DF
    v = _values(lib, alpha, band, need)
    w = _values(lib, alpha, band, need, fp64=1)
    err = 4e-6  # relative FP32 error bound of a statistic; four times it are to spare
    for df in range(1, CRIT_DF):
        x, y, x64, y64 = v[df]
        assert 0 < x64 < y64 and 0 <= x <= x64 and y >= y64
        assert chi2.sf(x64, df) > alpha > chi2.sf(y64, df)
        assert y64 / x64 < 1 + 1e-4  # no wider than it has to be
        assert x == 0.0 or chi2.sf(x * (1 + 4 * err), df) > alpha + band
        # (alpha = band: up to half an ulp of alpha)
        assert np.isinf(y) or chi2.sf(y * (1 - 4 * err), df) <= max(alpha - band, 1.1e-16 * alpha)
        assert (x == 0.0) == (alpha + band > 1 - 1e-9)
        assert np.isinf(y) == (alpha < band)
        if x > 0:  # (a part in 10^3 of the statistic covers both margins)
            assert chi2.sf(x * (1 + 1e-3), df) < alpha + band
        if alpha > band:
            assert chi2.sf(y * (1 - 1e-3), df) > alpha - band
        assert (w[df] == [x64, y64, x64, y64]).all()


@pytest.mark.parametrize("alpha", [1e-300, 1e-100, 1 - 1e-12])
def test_extreme_alphas_leave_every_decision_to_the_tail(lib, alpha):
    v = _values(lib, alpha, 1e-3, [1] * CRIT_DF)
    assert (v[:, [0, 2]] == 0).all() and np.isinf(v[:, [1, 3]]).all()


def test_only_reachable_df(lib):
    def needed(cards, adjusted):
        out = np.zeros(CRIT_DF, dtype=np.uint8)
        lib.needed(bytes(bytearray(int(c in cards) for c in range(6))), 5, adjusted, out.ctypes.data)
        return set(np.nonzero(out)[0].tolist())

    for cards in ([2], [1, 2, 3], [2, 3, 4], [3, 5], [2, 3, 4, 5]):
        r = [c for c in cards if c > 1]
        want = {(a - 1) * (b - 1) * c for a in r for b in r for c in [1] + r}
        assert needed(cards, 0) == want
        assert needed(cards, 1) == set(range(1, max(want) + 1))
    assert needed([1], 0) == set() and needed([], 1) == set()
    v = _values(lib, 0.05, 1e-3, [0] * CRIT_DF)
    assert (v[:, [0, 2]] == 0).all() and np.isinf(v[:, [1, 3]]).all()  # nothing certain
