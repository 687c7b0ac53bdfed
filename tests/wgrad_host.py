"""The weight-gradient plans of the block models (csrc/wgrad_plan.h, host arithmetic), as the library makes them."""
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TILES = ("192x384", "128x128", "128x128 two groups", "64x64 four groups")

DRIVER = r"""
#include <cstdio>
#include "wgrad_plan.h"
using namespace qsr;
// reads models (workers, tokens, width, hidden width, blocks, attention); a line for each launch: of one block's MLP (0) or attention
// half (1) or of all blocks (2), tile, ranges, tokens of a range, floats of partial results needed and held
int main()
{
    long long K, M, d, dh, L;
    int attention;
    while (scanf("%lld %lld %lld %lld %lld %d", &K, &M, &d, &dh, &L, &attention) == 6) {
        const bool all = wgrad_defer(K, M, d, dh, attention, L);
        const long long room = wgrad_split_floats(K, M, d, dh, attention, L, all);
        for (int what = all ? 2 : 0; what <= (all ? 2 : attention); ++what) {
            const WgradCover c = wgrad_cover(what != 1, all, K, d, dh, attention, L);
            const WgradPlan p = wgrad_plan_load(c.load, (int)M, 256, room, K * c.floats);
            printf("%lld %lld %lld %lld %lld %d  %d %d %d %d %lld %lld\n", K, M, d, dh, L, attention, what, (int)p.tile, p.split,
                   p.k_chunk, p.split * K * c.floats, room);
        }
    }
    return 0;
}
"""


def plans(models):
    """[(model, launch, tile, ranges, tokens of a range, floats needed, floats held)] of models (K, tokens, d, d_hidden, blocks, attention)."""
    with tempfile.TemporaryDirectory() as tmp:
        src, exe = os.path.join(tmp, "driver.cpp"), os.path.join(tmp, "driver")
        with open(src, "w") as f:
            f.write(DRIVER)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2310_14423_amd", "csrc"), src, "-o", exe],
                       check=True, timeout=120)
        out = subprocess.run([exe], input="\n".join("%d %d %d %d %d %d" % m for m in models), capture_output=True, text=True,
                             check=True, timeout=120).stdout
    rows = [tuple(map(int, l.split())) for l in out.splitlines()]
    return [(r[:6], ("mlp", "attention", "all")[r[6]], TILES[r[7]]) + r[8:] for r in rows]
