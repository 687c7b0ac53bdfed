"""The rows of the LayerNorm backward pass (csrc/ln_rows.h): every row belongs to a step and no partial row of the sums is without rows.  Few
rows: one step a wavefront, eight wavefronts to a partial row.  Else at least four rows a wavefront, each with a partial row of its own, and no
more wavefronts than the chip holds."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include <initializer_list>
#include "ln_rows.h"
int main()
{
    for (int K : {1, 2, 8, 16})
        for (int M : {1, 7, 63, 64, 100, 1040, 5885, 12608, 300001})
            for (int d = 64; d <= 1024; d += 64) {
                const qsr::LnBwdPlan q = qsr::ln_bwd_plan(K, M, d);
                printf("%d %d %d %d %d %lld\n", K, M, d, q.few ? 1 : 0, q.step, q.waves);
            }
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_no_wavefront_without_rows(tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2310_14423_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    rows = [tuple(map(int, l.split())) for l in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.splitlines()]
    assert len(rows) == 4 * 9 * 16
    seen = set()
    for K, M, d, few, step, waves in rows:
        side = 4 if d <= 64 else 2 if d <= 128 else 1                 # rows side by side in a wavefront
        slots = 256 * (20 if d <= 512 else 16 if d <= 768 else 12)    # wavefronts that the chip holds
        assert few == (K * M <= 4 * slots), (K, M, d)
        if few:
            assert step == side and (waves - 1) * 8 * step < M <= waves * 8 * step, (K, M, d)
        else:
            assert step % side == 0 and waves <= -(-M // step) and waves <= -(-M // 4), (K, M, d)
            assert K * waves <= K + slots, (K, M, d)
        seen.add((few, d))
    assert len(seen) == 2 * 16
