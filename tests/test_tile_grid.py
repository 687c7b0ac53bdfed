"""Grids of launches that number their tiles themselves (csrc/tile_grid.h): whole, no row of workgroups idle, and within what a launch
takes.  The perceptron's two gradients of 4 194 240 samples and 8130 hidden units are 8.4 million tiles of 64 x 64."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "tile_grid.h"
int main(int, char **argv)
{
    const qsr::TileGrid g = qsr::tile_grid(atoll(argv[1]), atoi(argv[2]));
    printf("%u %u\n", g.x, g.y);
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_all_tiles_within_the_limits(tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2310_14423_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    big = 128 * (1 + 65535) + 128                       # the sizes above
    for tiles in (1, 7, 1 << 22, (1 << 22) + 1, (1 << 23) - 1, 1 << 23, big, (1 << 31) - 1):
        for threads in (256, 512):
            x, y = map(int, subprocess.run([str(exe), str(tiles), str(threads)], capture_output=True, text=True, check=True).stdout.split())
            assert x * threads < 1 << 32 and 1 <= y <= 65536 and tiles <= x * y < tiles + x
    assert subprocess.run([str(exe), str(1 << 40), "512"], capture_output=True, text=True, check=True).stdout.split() == ["0", "0"]


def test_the_pair_of_products_takes_its_grid_from_there():
    """... and refuses no number of tiles that fits it."""
    code = open(os.path.join(ROOT, "paper_2310_14423_amd", "csrc", "sgemm.h")).read()
    body = code[code.index("hipError_t launch_sgemm_pair("):]
    body = body[:body.index("\n}")]
    assert "tile_grid(all" in body and "0x7FFFFFll" not in body
