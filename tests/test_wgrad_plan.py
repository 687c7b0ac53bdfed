"""The token ranges a launch of weight gradients of the block models is cut into, against the workspace carved for their
partial results (both host arithmetic, csrc/wgrad_plan.h): whatever the widths, one never exceeds the other."""
import itertools
import os
import shutil
import subprocess

import pytest

import wgrad_host

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


MANY_BLOCKS = r"""
#include <cstdio>
#include "wgrad_plan.h"
using namespace qsr;
int main()
{
    for (int attention = 0; attention < 2; ++attention)
        for (long long n : {2ll, 1000ll, 16383ll, 16384ll, 32767ll, 32768ll, 40000ll})
            printf("%d %lld %d\n", attention, n, (int)wgrad_defer(1, 64, 64, 64, attention, n));
    return 0;
}
"""


def _run(tmp_path, code):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(code)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2310_14423_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True, timeout=120)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
    return out


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_no_launch_of_all_blocks_beyond_the_grid(tmp_path):
    """The launches behind a shared weight-gradient launch have an entry along the grid's z extent (at most 65536) for every
    LayerNorm parameter of every block."""
    rows = [tuple(map(int, l.split())) for l in _run(tmp_path, MANY_BLOCKS).stdout.splitlines()]
    for attention, n_blocks, deferred in rows:
        assert not deferred or 2 * n_blocks * (1 + attention) + 1 <= 65536
    assert {n for _, n, deferred in rows if deferred} >= {2, 1000, 16383, 32767}      # as far as the grid goes


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_partial_results_fit_their_workspace():
    models = itertools.product((1, 2, 3, 5, 8, 16, 64), (1, 31, 1023, 1024, 1040, 4096, 4129, 12608, 1 << 20), range(64, 1025, 64),
                               (64, 128, 192, 512, 1024, 3072, 4608), (1, 2, 5, 12), (0, 1))
    cut, wide = {}, 0
    for (K, M, d, dh, L, attention), what, tile, ranges, chunk, need, room in wgrad_host.plans(models):
        # room for four ranges of this launch, of 256 MiB of them, or of none where the model's largest takes more than that in two
        largest = max(2 * d * dh + d + dh, attention * (4 * d * d + 4 * d)) if what != "all" else need // ranges // K
        assert room >= min(4 * (need // ranges), 1 << 26) or M < 1024 or 2 * K * (largest + 2 * d) > 1 << 26, (K, M, d, dh, L, attention, what)
        if ranges <= 1:
            continue
        cut[what, tile] = cut.get((what, tile), 0) + 1
        wide += dh < d and not attention
        assert ranges <= 4 and chunk % 32 == 0 and chunk * (ranges - 1) < M <= chunk * ranges, (K, M, d, dh, L, attention, what)
        assert need <= room, (K, M, d, dh, L, attention, what, tile, ranges, need, room)
    # every launch in every tile shape with ranges, and those of a model that is wider than its hidden layer
    assert len(cut) == 12 and min(cut.values()) >= 20 and wide > 100, (cut, wide)
