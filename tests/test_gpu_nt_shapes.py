"""GPU: the block models' gradients with every kind of output of the forward and data-gradient products in every tile shape that it takes
(test_nt_plan.py holds the cases to that), at the sizes where these go wrong if they do: last tiles of one row and one row short, a last panel of one, two and three tiles, rings longer than the contraction and
contractions of an odd and an even number of stages.  Against the oracle with the bf16 tolerances of test_gpu_parity.py."""
import numpy as np
import pytest

import workloads
from test_gpu_parity import VIT_TAIL, _assert_groups_close
from util import gpu_ctx, oracle_run

pytestmark = pytest.mark.gpu

CASES = [
    dict(d_in=64, d_hidden=192, B_loc=65, K=3),                                 # rings longer than contractions of two stages
    dict(d_in=320, d_hidden=448, B_loc=191, K=2),                               # last panels of one and of three tiles
    dict(d_in=192, d_hidden=576, B_loc=193, K=2, n_heads=3, seq_len=193),
    dict(d_in=128, d_hidden=3200, B_loc=257, K=2),                              # 100 stages through a ring of 8
    dict(d_in=256, d_hidden=640, B_loc=1153, K=7),                              # the last row tile holds one row
    dict(d_in=832, d_hidden=1664, B_loc=383, K=4),                              # and one row short; an odd number of stages
    dict(d_in=512, d_hidden=1088, B_loc=769, K=8),
    dict(d_in=256, d_hidden=1088, B_loc=1281, K=8),
    dict(d_in=320, d_hidden=1088, B_loc=3073, K=8),
    dict(d_in=1024, d_hidden=1024, B_loc=1025, K=8),                            # the widest: 256 x 256 in all products but the loss's
    # each kind of output in the shapes that the ones above leave out
    dict(d_in=448, d_hidden=64, B_loc=127, K=5),
    dict(d_in=768, d_hidden=64, B_loc=129, K=32),
    dict(d_in=896, d_hidden=64, B_loc=257, K=32),
    dict(d_in=576, d_hidden=384, B_loc=513, K=32),
    dict(d_in=64, d_hidden=128, B_loc=513, K=32, n_heads=1, seq_len=171),
    dict(d_in=128, d_hidden=128, B_loc=513, K=32, n_heads=2, seq_len=171),
    dict(d_in=192, d_hidden=64, B_loc=2049, K=24, n_heads=3, seq_len=3),
    dict(d_in=448, d_hidden=64, B_loc=513, K=32, n_heads=7, seq_len=171),
]


@pytest.mark.parametrize("dims", CASES)
def test_gradient_by_product_shape(dims):
    heads = dims.get("n_heads", 0)
    w = workloads.get("vit" if heads else "resmlp", T=4, T_warm=1, n_blocks=1, **dims)
    th0 = workloads.theta0(w)
    th0 = (th0 + 0.02 * np.random.default_rng(3).standard_normal(th0.size)).astype(np.float32)
    ctx = gpu_ctx(w, theta0=th0)
    orc = oracle_run(w, theta0=th0)
    ctx.local_step()
    g, loss = ctx.grads.cpu().numpy(), ctx.read_loss()
    ctx.close()
    for k in {0, dims["K"] - 1}:
        want_g, wl = orc.grad(k, 0, th0.astype(np.float64))
        assert loss[k] == pytest.approx(wl, rel=1e-2)
        if heads:
            _assert_groups_close(w, g[k], want_g, "shape k=%d" % k, tail=VIT_TAIL, weights_only_tail=True)
        else:
            _assert_groups_close(w, g[k], want_g, "shape k=%d" % k, tail=(1e-5, 1.5))
