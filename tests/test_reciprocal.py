"""Division by reciprocals (lpp_reciprocal.h), tried on the host: the header the kernels include, compiled as plain C++ (no GPU)."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_06352_amd", "csrc")
SOURCE = """
#include "lpp_reciprocal.h"
extern "C" uint32_t by_rc(uint32_t n, uint32_t d) { return div_rc(n, d, reciprocal(d)); }
extern "C" uint32_t by_either(uint32_t n, uint32_t d, uint64_t most) { return div_or_rc(n, d, reciprocal(d, most)); }
extern "C" int32_t layers(int64_t units, int32_t most) { return layers_per_launch(units, most); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("reciprocal")
    (d / "t.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", "/opt/rocm/include",
                    str(d / "t.cpp"), "-o", str(d / "t.so")], check=True)
    L = C.CDLL(str(d / "t.so"))
    L.by_rc.argtypes, L.by_rc.restype = [C.c_uint32] * 2, C.c_uint32
    L.by_either.argtypes, L.by_either.restype = [C.c_uint32, C.c_uint32, C.c_uint64], C.c_uint32
    L.layers.argtypes, L.layers.restype = [C.c_int64, C.c_int32], C.c_int32
    return L


def _around(d, most):
    return {n for m in range(0, most + d, d) for n in (m - 1, m, m + 1) if 0 <= n < most}


@pytest.mark.parametrize("units", [1, 7, 768, 3072, 16376, 16383, 16384, 16385, 16640, 17000, 20480, 24000, 30000, 46000, 1 << 20, (1 << 27) + 8])
def test_units_of_a_launch_find_their_layer(lib, units):
    # a launch's last units of each layer: 16 layers of 16640 units and more had one that was given to the layer behind it
    most = lib.layers(units, 16)
    assert 1 <= most <= 16 and (most == 16 or units > 16383)
    if most > 1:                                            # (one layer: not divided)
        assert all(lib.by_rc(n, units) == n // units for n in _around(units, units * most))
    if units in (16640, 20480, 30000):
        assert any(lib.by_rc(n, units) != n // units for n in _around(units, units * 16))


@pytest.mark.parametrize("d", [1, 2, 3, 7, 8, 20, 24, 61, 1000, 65535])
def test_numbers_below_the_bound_and_beyond(lib, d):
    for n in [0, 1, d - 1, d, d + 1, 10 * d - 1, 10 * d] + [x + e for x in (2 ** 32 // d, 2 ** 32 // d // 2) for e in (-2, -1)]:
        if 0 <= n and n * d < 2 ** 32:
            assert lib.by_rc(n, d) == n // d
    for n in (2 ** 31 - 1, 2 ** 32 - 1, (2 ** 32 - 1) // d * d, (2 ** 32 - 1) // d * d - 1):
        assert lib.by_either(n, d, 2 ** 32 - 1) == n // d
