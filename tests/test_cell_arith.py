"""FP64 quotients of the cell updates (csrc/mg_arith.h, compiled for the host)
against divisions, with a reciprocal as far off as the hardware's."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2110_00328_amd", "csrc")
SHIM = r"""
#include "mg_arith.h"
#include <cstdint>
#include <random>
using namespace mgg;

// number of x with sixth(x) != x / 6
extern "C" int64_t sixths_off(int64_t m, int seed) {
  std::mt19937_64 g(seed);
  std::uniform_real_distribution<double> lg(-60.0, 60.0);
  int64_t off = 0;
  for (int64_t i = 0; i < m; ++i) {
    const double x = (i & 1 ? -1.0 : 1.0) * std::exp(lg(g));
    off += sixth(x) != x / 6.0;
  }
  return off;
}

// number of (a, b) with quotient(a, b) != a / b, the reciprocal off by up to d
extern "C" int64_t quotients_off(int64_t m, int seed, double d) {
  std::mt19937_64 g(seed);
  std::uniform_real_distribution<double> lg(-60.0, 60.0), one(-1.0, 1.0);
  int64_t off = 0;
  for (int64_t i = 0; i < m; ++i) {
    const double a = (i & 1 ? -1.0 : 1.0) * std::exp(lg(g)), b = std::exp(lg(g));
    const double k = 1.0 + d * one(g);
    off += quotient(a, b, [k](double x) { return k / x; }) != a / b;
  }
  return off;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("cell_arith")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "shim.so")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-Wall", "-Werror",
                           "-shared", "-fPIC", "-I", CSRC, "-o", so, str(d / "shim.cpp")])
    lib = ctypes.CDLL(so)
    lib.sixths_off.restype = lib.quotients_off.restype = ctypes.c_int64
    lib.sixths_off.argtypes = [ctypes.c_int64, ctypes.c_int]
    lib.quotients_off.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_double]
    return lib


def test_a_sixth_is_the_division(lib):
    assert lib.sixths_off(2000000, 1) == 0


# a quotient could round otherwise only within 2^-88 of the middle between two
# numbers: none of these
@pytest.mark.parametrize("d", [0.0, 2.0 ** -29, 2.0 ** -22])
def test_quotients_are_divisions(lib, d):
    assert lib.quotients_off(2000000, 2, d) == 0
