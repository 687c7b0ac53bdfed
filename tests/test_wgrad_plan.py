"""The token ranges a weight gradient of the block models is cut into, against the workspace carved for their
partial results (both host arithmetic, csrc/wgrad_plan.h): whatever the widths, one never exceeds the other."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include <initializer_list>
#include "wgrad_plan.h"
using namespace qsr;
int main()
{
    long long cut = 0, wide = 0;
    const int tokens[] = {1, 31, 4095, 4096, 4129, 5000, 12608, 1 << 20};
    for (int K : {1, 2, 3, 5, 8, 16, 64})
        for (int d = 64; d <= 1024; d += 64)
            for (int dh : {64, 128, 192, 256, 512, 768, 1024, 2048, 3072, 4608})
                for (int attention = 0; attention < 2; ++attention) {
                    const WgradSpace sp = wgrad_space(K, d, dh, attention);
                    const int mn[4][2] = {{d, dh}, {dh, d}, {d, 3 * d}, {d, d}};
                    for (int i = 0; i < (attention ? 4 : 2); ++i)
                        for (int t : tokens) {
                            const long long M = mn[i][0], N = mn[i][1];
                            const WgradPlan p = wgrad_plan(M, N, t, K, 256);
                            if (p.split <= 1) continue;
                            ++cut;
                            wide += dh < d && !attention;
                            const bool ranges = p.split <= WGRAD_SPLIT && p.k_chunk % 32 == 0 &&
                                                (long long)p.k_chunk * p.split >= t && (long long)p.k_chunk * (p.split - 1) < t;
                            if (!ranges || K * p.split * M * N > sp.products || K * p.split * N > sp.biases) {
                                printf("K=%d d=%d dh=%d attention=%d %lldx%lld tokens=%d split=%d\n", K, d, dh, attention, M, N, t, p.split);
                                return 1;
                            }
                        }
                }
    printf("%lld %lld\n", cut, wide);
    return 0;
}
"""


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
def test_partial_results_fit_their_workspace(tmp_path):
    out = _run(tmp_path, DRIVER)
    cut, wide = map(int, out.stdout.split())
    assert cut > 1000 and wide > 100          # the cut ones, and those of a model that is wider than its hidden layer
