"""The tile shapes of the block models' forward and data-gradient products (csrc/nt_plan.h, host arithmetic), as the library takes them."""
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHAPES = ("64x64", "64x64 long", "128x128", "128x128 long", "128x256", "256x256")
OUTPUTS = ("gelu", "factor", "residual", "bf16", "f32", "loss")

DRIVER = r"""
#include <cstdio>
#include "nt_plan.h"
using namespace qsr;
// reads products (output, M, N, K, batch); the shape, its tiles, and the estimates of all
int main()
{
    int out;
    long long M, N, K, batch;
    while (scanf("%d %lld %lld %lld %lld", &out, &M, &N, &K, &batch) == 5) {
        const NtShape s = nt_shape((NtOut)out, M, N, K, batch, 256);
        printf("%d %lld", (int)s, nt_tiles(s, M, N, batch));
        for (int i = 0; i < NT_SHAPES; ++i) printf(" %.17g", nt_us((NtShape)i, (NtOut)out, nt_tiles((NtShape)i, M, N, batch), K, 256));
        printf("\n");
    }
    return 0;
}
"""


def shapes(products):
    """[(shape, tiles, estimates in us)] of products (output, M, N, K, batch)."""
    with tempfile.TemporaryDirectory() as tmp:
        src, exe = os.path.join(tmp, "driver.cpp"), os.path.join(tmp, "driver")
        with open(src, "w") as f:
            f.write(DRIVER)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2310_14423_amd", "csrc"), src, "-o", exe],
                       check=True, timeout=120)
        text = "\n".join("%d %d %d %d %d" % ((OUTPUTS.index(p[0]),) + tuple(p[1:])) for p in products)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=120).stdout
    rows = [l.split() for l in out.splitlines()]
    return [(SHAPES[int(r[0])], int(r[1]), [float(v) for v in r[2:]]) for r in rows]


def model_products(d, dh, heads, tokens, K):
    """The forward and data-gradient products of a block model, in the order of a pass: (what, output, M, N, K, batch)."""
    attn = [("qkv", "bf16", 3 * d, d), ("projection", "residual", d, d)] if heads else []
    back = [("projection gradient", "bf16", d, d), ("qkv gradient", "f32", d, 3 * d)] if heads else []
    rows = attn + [("gelu", "gelu", dh, d), ("second", "residual", d, dh), ("loss", "loss", d, d), ("gelu gradient", "factor", dh, d),
                   ("first gradient", "f32" if heads else "bf16", d, dh)] + back
    return [(what, out, tokens, n, k, K) for what, out, n, k in rows]
