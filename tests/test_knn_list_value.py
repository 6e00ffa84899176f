"""The ordering bound of the neighbour build's list words, tried on the host: the header the kernels include,
compiled as plain C++ (no GPU).  Values further apart than ``list_margin`` must belong to similarities further
apart than twice the error they were given."""
import ctypes as C
import os
import subprocess
from fractions import Fraction

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_06352_amd", "csrc")
SOURCE = """
#include "lpp_knn_list.h"
extern "C" void values(const int32_t* d, int n, float a, uint32_t qmax, uint32_t* v) {
  for (int i = 0; i < n; ++i) v[i] = list_value((float)d[i], a, qmax);
}
extern "C" int32_t margin(double e, double range, uint32_t qmax) { return list_margin(e, range, qmax); }
extern "C" double apart(float reach, int32_t D) { return key_margin(reach, D); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("knn_list")
    (d / "t.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-ffp-contract=off", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", CSRC,
                    "-I", "/opt/rocm/include", str(d / "t.cpp"), "-o", str(d / "t.so")], check=True)
    L = C.CDLL(str(d / "t.so"))
    L.values.argtypes = [C.c_void_p, C.c_int, C.c_float, C.c_uint32, C.c_void_p]
    L.margin.argtypes = [C.c_double, C.c_double, C.c_uint32]
    L.margin.restype = C.c_int32
    L.apart.argtypes = [C.c_float, C.c_int32]
    L.apart.restype = C.c_double
    return L


# value bits: 24 (codebooks of up to 256 codes) down to 16 (65536 codes)
@pytest.mark.parametrize("bits", [24, 23, 22, 21, 20, 19, 16])
def test_values_beyond_the_margin_are_ordered(lib, bits):
    g = np.random.default_rng(bits)
    qmax = (1 << bits) - 2
    worst = 0
    for scale in (0.004, 0.02, 0.3, 1.0):                   # list units per integer unit of the similarity
        rng = int(qmax / scale)
        a = float(np.float32(qmax / rng))
        for gap in (1, 2, 3, 10, 100, 1000):                # 2 e: similarities this close may be in either order
            m = lib.margin(gap / 2.0, float(rng), qmax)
            lo = g.integers(0, max(rng - gap, 1), size=20000).astype(np.int32)
            lo[:4000] = max(rng - gap, 1) - 1 - np.arange(4000) % max(rng // 2, 1)    # the largest round the most
            lo = np.maximum(lo, 0)
            v = []
            for d in (lo, lo + np.int32(gap)):
                d = np.ascontiguousarray(d, dtype=np.int32)
                out = np.empty(len(d), dtype=np.uint32)
                lib.values(d.ctypes.data, len(d), a, qmax, out.ctypes.data)
                v.append(out.astype(np.int64))
            worst = max(worst, int((v[1] - v[0]).max()) - m)
    assert worst <= 0, f"values of similarities inside the error differ by {worst} more than the margin"


def test_margin_is_not_wasteful(lib):
    # at 19 bits and fewer the rounding term is below one unit
    assert lib.margin(0.0, 1000.0, (1 << 19) - 2) == 1
    assert lib.margin(5.0, 1000.0, 1000) in (11, 12)
    assert lib.margin(float("nan"), 1.0, 1000) == lib.margin(1e300, 1e-3, 1000) == 1 << 30


# vanishing: numbers whose squares float32 does not hold beside one that it just does; large: products near its end
@pytest.mark.parametrize("kind", ["unit", "vanishing", "large", "one"])
@pytest.mark.parametrize("D", [17, 96, 256])
def test_sums_beyond_the_margin_have_the_order_of_the_keys(lib, D, kind):
    # four times the error that any order of a sum can have, by the exact sum of the magnitudes, stays below the margin,
    # and two ways of adding differ by far less
    g = np.random.default_rng(D)
    rows, codes = g.standard_normal((2, 40, D)).astype(np.float32)
    if kind == "vanishing":
        rows = np.full((40, D), 2.6e-23, dtype=np.float32)
        rows[:, 0] = 4e-23
        codes = (codes * 1e9).astype(np.float32)
        codes[:20] = np.float32(1e9)
    elif kind == "large":
        rows, codes = rows * np.float32(1e17), codes * np.float32(1e17)
    elif kind == "one":
        rows[:, 1:] = 0
    mabs = np.abs(codes).max()
    for x in rows:
        l1 = np.float32(0)
        for v in np.abs(x):
            l1 = np.float32(l1 + v)
        apart = lib.apart(float(np.float32(l1 * mabs)), D)
        for y in codes:
            products = [Fraction(float(a)) * Fraction(float(b)) for a, b in zip(x, y)]
            assert 4 * D * Fraction(1, 2 ** 53) * sum(abs(p) for p in products) <= Fraction(apart)
            key = lanes = 0.0
            for p in products:
                key += float(p)                             # (exact: 48 bits)
            for i in range(16):
                part = 0.0
                for p in products[i::16]:
                    part += float(p)
                lanes += part
            assert abs(key - lanes) <= apart / 2
