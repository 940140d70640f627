"""The layout of tiled launches covers every ray of a run once, at every size a
run can have: one ray, ragged rows, and more rays than 32-bit counts of tiles
hold (a part of a run, or a source without strata, is a single row of tiles)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2410_08747_amd", "csrc")


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("tiles") / "tile_layout")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, os.path.join(HERE, "tile_layout.cpp"), "-o", exe],
                   check=True)
    return lambda *case: subprocess.run([exe], input=" ".join(str(x) for x in case), capture_output=True, text=True,
                                        check=True).stdout.strip()


@pytest.mark.parametrize("first,n,rows,ratio", [
    (0, 1, 1, 1.0), (5, 257, 1, 1.0), (0, 15, 1, 1.0), (0, 1023, 3, 1.0), (0, 99_991, 37, 1.0), (0, 1_000_003, 250, 1.0),
    (17, 4_000_037, 500, 0.02), (17, 4_000_037, 500, 60.0)])
def test_every_ray_once(layout, first, n, rows, ratio):
    assert layout(first, n, rows, ratio) == "ok"


@pytest.mark.parametrize("rows", [1, 37, 4096])
@pytest.mark.parametrize("n", [(1 << 23) + 12_345, 10**9, (1 << 44) - 1, 1 << 44, (1 << 44) + 4097, 2 * 10**13, (1 << 51) + 3])
def test_large_runs(layout, n, rows):
    assert layout(0, n, rows, 1.0) == "ok"
    assert layout(n // 3, n, rows, 1.0) == "ok"
