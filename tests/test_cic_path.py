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
extern "C" int prefers_binned(int n, int64_t np) { return mgg::cic_prefers_binned(n, np); }
extern "C" int makes_both(int n) { return mgg::cic_makes_both(n); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("cic_path")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "shim.so")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC",
                           "-I", CSRC, "-o", so, str(d / "shim.cpp")])
    lib = ctypes.CDLL(so)
    lib.prefers_binned.argtypes = [ctypes.c_int, ctypes.c_int64]
    return lib


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


# cells a side, particles, us of binned and direct deposits in grid order, then
# in no order (MI355X; medians, which repeat to 2%)
TIMES = [
    (32, 1000, 20.0, 11.0, 21.1, 11.3), (32, 64000, 63.4, 20.2, 103.1, 28.5),
    (32, 1061208, 613.0, 283.4, 1370.7, 367.4), (48, 64000, 43.8, 22.2, 62.3, 29.7),
    (48, 262144, 74.4, 71.0, 138.6, 99.4), (48, 531441, 113.4, 131.9, 273.3, 194.8),
    (48, 2097152, 399.2, 473.7, 968.8, 743.7), (64, 32768, 25.0, 17.3, 31.0, 19.0),
    (64, 132651, 43.4, 42.5, 61.6, 54.7), (64, 262144, 51.7, 68.5, 87.0, 97.4),
    (64, 1061208, 112.2, 266.3, 266.9, 369.8), (96, 32768, 24.5, 20.5, 28.2, 21.3),
    (96, 64000, 25.2, 29.5, 30.4, 32.3), (96, 132651, 26.8, 50.7, 40.1, 57.7),
    (128, 32768, 26.1, 25.0, 29.7, 25.4), (128, 64000, 27.0, 35.1, 32.1, 36.4),
    (160, 32768, 29.8, 31.5, 34.4, 32.1), (192, 8000, 38.5, 32.7, 42.0, 32.8),
    (192, 32768, 38.1, 39.8, 43.8, 40.6), (256, 1000, 50.3, 58.5, 48.6, 58.6),
    (256, 64000, 57.9, 76.5, 64.8, 76.5), (384, 1000, 97.0, 258.9, 96.1, 258.6),
    (384, 64000, 130.6, 288.2, 142.5, 288.4), (512, 8000, 264.8, 599.9, 263.4, 599.0),
    (512, 132651, 282.9, 660.8, 296.4, 663.0), (512, 2097152, 359.1, 1370.8, 533.9, 1421.8),
    (50, 262144, 70.8, 68.4, 125.1, 97.7), (50, 531441, 104.7, 130.6, 241.8, 191.8),
    (50, 2097152, 354.3, 497.7, 863.8, 729.4), (58, 262144, 56.9, 69.6, 99.1, 97.9),
    (58, 531441, 80.6, 134.2, 181.3, 192.4), (62, 132651, 44.5, 42.0, 65.0, 56.0),
    (62, 262144, 54.9, 70.0, 90.4, 97.7), (72, 132651, 42.8, 44.3, 58.0, 55.0),
    (72, 262144, 49.3, 72.6, 78.7, 98.0), (82, 64000, 26.9, 28.1, 33.8, 30.9),
    (90, 64000, 25.4, 29.2, 31.2, 31.6), (100, 64000, 28.0, 30.6, 32.6, 32.3),
    (100, 132651, 29.6, 51.1, 42.6, 57.8), (140, 32768, 29.9, 27.3, 33.7, 27.7),
    (200, 32768, 45.7, 42.4, 51.2, 42.5), (200, 64000, 46.7, 53.1, 53.0, 53.1),
    (200, 1061208, 61.3, 351.5, 173.5, 395.3), (250, 8000, 67.3, 55.7, 67.5, 55.9),
    (250, 32768, 63.5, 63.3, 69.9, 63.3), (300, 8000, 94.3, 98.2, 94.0, 99.7),
    (300, 132651, 93.8, 141.6, 106.2, 144.3)]


@pytest.mark.parametrize("row", TIMES, ids=lambda r: f"{r[0]}-{r[1]}")
def test_choice_agrees_with_measured_times(lib, row):
    n, count, *us = row
    binned = lib.prefers_binned(n, count)
    for b, d in (us[:2], us[2:]):
        # at most 3% above the path that ran whatever the particles before
        # there was a choice: binned on whole tiles, direct on other sides
        assert (b if binned else d) <= 1.03 * (d if n % 16 else b)
    if n % 16 == 0:  # and never the slower one by that much in both orders
        (b0, d0), (b1, d1) = us[:2], us[2:]
        if binned:
            assert b0 <= 1.03 * d0 or b1 <= 1.03 * d1
        else:
            assert d0 <= 1.03 * b0 or d1 <= 1.03 * b1


# more particles never turn a deposit back to the direct path
@pytest.mark.parametrize("n", [16, 32, 48, 50, 58, 64, 66, 200, 256, 300, 512, 1600])
def test_choice_changes_once_with_the_number_of_particles(lib, n):
    picks = [lib.prefers_binned(n, int(1.2 ** e)) for e in range(122)]
    assert picks == sorted(picks)
