"""The size rules of the 2D dispatch (plain C++), compiled on the CPU: each
listed grid takes the kernel that measured faster on 256 compute units."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1212_0204_amd", "csrc")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "r.cpp").write_text('''#include "rules.hpp"
extern "C" int tiles(int nx, int ny, int ncu) { return hofks::euler_tiles(nx, ny, ncu); }
extern "C" int pairs(int nx, int ny, int ncu) { return hofks::offlattice_pairs(nx, ny, ncu); }
extern "C" int rows(int nx, int ny, int nv, int fp32, int ncu) {
  return hofks::strip_rows(nx, ny, nv, fp32, ncu);
}
extern "C" int wavefronts(int nx, int ny, int nv, int ncu) {
  return hofks::fp32_wavefronts(nx, nv, (long)((nx + 63) / 64) * ny, ncu);
}
''')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "r.so"),
                    str(d / "r.cpp")], check=True)
    return ctypes.CDLL(str(d / "r.so"))


@pytest.mark.parametrize("n,tiles", [
    ((4, 4096), 1), ((8, 8192), 1), ((16, 4096), 1), ((16, 16384), 1), ((20, 3276), 1), ((32, 2048), 1),
    ((32, 4096), 1), ((64, 1024), 1), ((64, 2048), 1), ((24, 5461), 1), ((32, 8192), 1),
    # few strips, lanes mostly busy, or several rounds of them
    ((8, 1024), 0), ((16, 1024), 0), ((32, 1024), 0), ((64, 512), 0), ((40, 1638), 0), ((48, 5461), 0),
    ((72, 910), 0), ((122, 537), 0), ((20, 13107), 0), ((64, 8192), 0), ((70, 37), 0), ((256, 256), 0),
    ((512, 512), 0), ((20000, 1), 0), ((4096, 4), 0)])
def test_euler_tiles_on_narrow_grids(rules, n, tiles):
    assert rules.tiles(n[0], n[1], 256) == tiles


@pytest.mark.parametrize("n,nv,w", [
    ((256, 256), 32, 2), ((300, 256), 32, 2), ((330, 300), 32, 4), ((200, 120), 32, 4),
    ((400, 400), 32, 8), ((512, 512), 32, 8), ((330, 853), 16, 8), ((200, 1024), 16, 8),
    ((70, 3840), 24, 8), ((512, 2048), 32, 8), ((128, 3840), 40, 8),
    # wavefronts without work enough in blocks of eight
    ((4, 20000), 8, 4), ((16, 5120), 16, 4), ((48, 5120), 24, 4), ((16, 3072), 32, 4), ((16, 4096), 64, 4),
    ((200, 1280), 8, 4), ((400, 1462), 8, 4), ((512, 960), 16, 4), ((128, 5120), 16, 4),
    ((128, 5120), 24, 4)])
def test_fp32_wavefronts(rules, n, nv, w):
    assert rules.wavefronts(n[0], n[1], nv, 256) == w


@pytest.mark.parametrize("n,fp64,fp32", [
    ((70, 37), 1, 1), ((256, 256), 1, 1), ((320, 300), 1, 1),
    # past two blocks of one row per compute unit
    ((320, 343), 1, 3), ((200, 550), 1, 3), ((256, 512), 1, 3), ((350, 350), 1, 3),
    ((72, 1527), 1, 3), ((128, 1024), 1, 2), ((122, 1074), 1, 2),  # a quarter of the lanes idle
    ((400, 400), 3, 3), ((364, 467), 4, 2), ((450, 450), 4, 2),
    ((512, 512), 5, 5), ((1000, 1000), 5, 5)])
def test_rows_per_strip(rules, n, fp64, fp32):
    assert (rules.rows(n[0], n[1], 24, 0, 256), rules.rows(n[0], n[1], 24, 1, 256)) == (fp64, fp32)


@pytest.mark.parametrize("n,nv,rows", [
    ((398, 332), 32, 3), ((396, 336), 32, 3), ((398, 332), 24, 1), ((385, 298), 32, 1),
    ((382, 336), 32, 1), ((72, 1527), 32, 1), ((300, 250), 32, 1)])
def test_rows_per_strip_beside_long_kinetic_launches(rules, n, nv, rows):
    assert rules.rows(n[0], n[1], nv, 0, 256) == rows


@pytest.mark.parametrize("n,pairs", [
    ((256, 256), 1), ((230, 256), 1), ((384, 256), 1), ((360, 400), 1), ((450, 128), 1), ((100, 400), 1),
    ((370, 198), 1), ((323, 194), 1), ((273, 212), 1), ((332, 371), 1),
    ((70, 37), 0), ((64, 64), 0), ((150, 150), 0), ((128, 256), 0), ((450, 64), 0), ((300, 128), 0),
    ((150, 400), 0), ((192, 400), 0), ((256, 400), 0), ((131, 375), 0), ((295, 197), 0), ((296, 393), 0), ((64, 4096), 0), ((300, 300), 0)])
def test_offlattice_in_the_two_cell_kernel(rules, n, pairs):
    assert rules.pairs(n[0], n[1], 256) == pairs
