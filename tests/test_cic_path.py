"""The choice between the two deposit paths (host code, csrc/cic_path.h)."""
import ctypes
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2110_00328_amd", "csrc")
SHIM = """
#include "cic_path.h"
extern "C" int takes_binned(int w, int b, int d, int c) { return mgg::cic_takes_binned(w, b, d, c); }
extern "C" int makes_both(int n) { return mgg::cic_makes_both(n); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("cic_path")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "shim.so")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC",
                           "-I", CSRC, "-o", so, str(d / "shim.cpp")])
    return ctypes.CDLL(so)


class Buffers:
    """What a context holds: the deposits of cic_assign with nothing but their buffers."""

    def __init__(self, lib, n, threshold):
        self.lib, self.n, self.threshold = lib, n, threshold
        self.binned_np, self.direct = 0, False

    def deposit(self, count, capturing):
        """the number of allocations"""
        took = 0
        binned = self.lib.takes_binned(int(count >= self.threshold), int(self.binned_np >= count),
                                       int(self.direct), int(capturing))
        if not self.direct and (not binned or self.lib.makes_both(self.n)):
            self.direct, took = True, took + 1
        if binned and self.binned_np < count:
            self.binned_np, took = count, took + 1
        return took


# whatever the path preferred from some number of particles on: a deposit
# under capture allocates nothing after one of as many particles, nor, on sides
# of no multiple of 16, after any; outside of one the first half holds too
@pytest.mark.parametrize("n", [32, 34, 512, 250])
def test_later_deposits_find_their_buffers(lib, n):
    rng = random.Random(n)
    for _ in range(2000):
        ctx = Buffers(lib, n, rng.choice([0, 10, 1000, 10 ** 9]))
        most = 0
        for _ in range(rng.randint(1, 6)):
            count, capturing = rng.randint(1, 2000), most > 0 and rng.random() < 0.5
            took = ctx.deposit(count, capturing)
            if count <= most or (capturing and n % 16):
                assert took == 0, (count, most, capturing)
            if not capturing:
                most = max(most, count)


def test_preferred_path_runs_when_its_buffers_can_be_made(lib):
    for have_direct in (0, 1):
        for have_binned in (0, 1):
            assert lib.takes_binned(1, have_binned, have_direct, 0) == 1
    assert lib.takes_binned(0, 0, 0, 0) == 0 and lib.takes_binned(0, 1, 1, 0) == 0
