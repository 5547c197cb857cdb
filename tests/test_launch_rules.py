"""The choice of wavefronts per work item (csrc/launch_rules.h), compiled for the host: an item
that one wavefront takes in about one go never gets more of them, however small the launch;
longer items do, up to launches that grow with their length; and the choices at sizes that
were measured on both sides of the line."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
#include "launch_rules.h"
extern "C" {
int pixels(int fp64, double groups, long n) { return celmi::wide_pixels(fp64, groups, n) ? celmi::kWideWaves : 1; }
int maps(int fp64, long n) { return celmi::wide_maps(fp64, n); }
int hessian(double passes, long n) { return celmi::hessian_waves(passes, n); }
long groups(long n, long item, long group) { return celmi::patch_groups(n, item, group); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("rules")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_1803_00113_amd", "csrc"),
                    str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    l = C.CDLL(str(d / "shim.so"))
    l.pixels.argtypes = [C.c_int, C.c_double, C.c_long]
    l.maps.argtypes = [C.c_int, C.c_long]
    l.hessian.argtypes = [C.c_double, C.c_long]
    l.groups.argtypes = [C.c_long, C.c_long, C.c_long]
    l.groups.restype = C.c_long
    return l


@pytest.mark.parametrize("length", [0.1, 0.44, 0.87, 1.0])
@pytest.mark.parametrize("n", [1, 20, 256, 1000, 4096])
def test_short_items_keep_one_wavefront(rules, length, n):
    assert rules.pixels(0, length, n) == 1 and rules.pixels(1, length, n) == 1 and rules.hessian(length, n) == 1


@pytest.mark.parametrize("length", [1.7, 2.5, 3.3, 6.5, 13.0, 100.0])
def test_launches_of_longer_items(rules, length):
    for f in (lambda n: rules.pixels(0, length, n), lambda n: rules.pixels(1, length, n), lambda n: rules.hessian(length, n)):
        got = [f(n) for n in (1, 64, 256, 512, 1024, 2048, 4096, 8192, 65536)]
        assert got[0] > 1 and got[-1] == 1 and got == sorted(got, reverse=True)


def test_measured_sizes(rules):
    """(length, items, several better) well off the crossover"""
    for length, n, wide in [(1.7, 645, 1), (1.7, 1300, 1), (1.7, 2670, 0), (2.5, 1815, 1), (2.5, 7725, 0), (3.3, 115, 1),
                            (3.3, 3610, 1), (3.3, 10950, 0), (6.1, 1915, 1)]:
        assert (rules.pixels(0, length, n) > 1) == bool(wide), (length, n)
    for length, n, wide in [(1.7, 250, 1), (1.7, 1060, 0), (3.3, 550, 1), (3.3, 1750, 1), (3.3, 3425, 0), (12.0, 1805, 1)]:
        assert (rules.pixels(1, length, n) > 1) == bool(wide), (length, n)
    for passes, n, waves in [(1.7, 440, 4), (1.7, 1265, 1), (3.4, 225, 4), (3.4, 1300, 4), (3.4, 5155, 1), (5.0, 875, 4),
                             (5.0, 3500, 1), (6.5, 115, 8), (6.5, 425, 8), (6.5, 665, 4), (6.5, 1985, 4), (6.5, 7650, 1),
                             (12.0, 185, 8), (12.0, 725, 4), (12.0, 3110, 4)]:
        assert rules.hessian(passes, n) == waves, (passes, n)
    assert rules.maps(0, 20) and not rules.maps(0, 5850) and rules.maps(1, 465) and not rules.maps(1, 2395)


@pytest.mark.parametrize("item", [64, 100, 128, 200, 512, 1024])
@pytest.mark.parametrize("group", [64, 128, 256])
def test_groups_are_counted_whole(rules, item, group):
    for n in (1, 63, 64, 65, 99, 128, 144, 200, 201, 512, 700, 1024, 2049):
        assert rules.groups(n, item, group) == sum(-(-min(item, n - b) // group) for b in range(0, n, item)), n


def test_items_of_a_group_and_a_bit(rules):
    """144 pixels are two passes of 128: 40 sources' 250 items in double precision (25.5 us by one
    wavefront, 16.9 by several) get several"""
    assert rules.pixels(1, rules.groups(144, 512, 128), 250) > 1
