"""GPU: the block models' gradients at narrow widths, many and few tokens, and at the sizes where the weight gradients change their tile shape
or split (the other products' shapes: test_gpu_nt_shapes.py), against the oracle with the bf16 tolerances of test_gpu_parity.py (which also says where they come from)."""
import numpy as np
import pytest

import wgrad_host
import workloads
from test_gpu_parity import VIT_TAIL, _assert_groups_close
from util import gpu_ctx, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [
    # contractions of two stages, into outputs 16 times as wide and ragged rows; of 32 stages into one tile's width
    dict(d_in=64, d_hidden=1024, n_blocks=1, B_loc=700, K=4),
    # a hidden layer 64 times as wide as the model
    dict(d_in=64, d_hidden=4096, n_blocks=1, B_loc=1021, K=8),
    # 192 columns: three tiles of 64, one and a half of 128; many tokens
    dict(d_in=192, d_hidden=64, n_blocks=1, B_loc=4000, K=8),
    dict(d_in=192, d_hidden=64, n_blocks=1, B_loc=6100, K=8),
    # weight gradients on 128 x 128 tiles with two groups (128 of them), a short token count for both groups
    dict(d_in=64, d_hidden=2048, n_blocks=1, B_loc=300, K=8),
    # weight gradients on 64 x 64 tiles with four groups, cut into four ranges, the last one ragged
    dict(d_in=64, d_hidden=128, n_blocks=1, B_loc=4129, K=2),
    # the same tiles, in one range; a hidden layer 72 times as wide as the model
    dict(d_in=64, d_hidden=4608, n_blocks=1, B_loc=4100, K=4),
    # a hidden layer narrower than the model: the second weight's gradient has more columns than any other's, cut into ranges
    dict(d_in=192, d_hidden=64, n_blocks=1, B_loc=4129, K=2),
    # fewer tokens than a stage
    dict(d_in=64, d_hidden=64, n_blocks=1, B_loc=7, K=1),
])
def test_gradient_where_the_tile_shape_changes(dims):
    w = workloads.get("resmlp", T=4, T_warm=1, **dims)
    rng = np.random.default_rng(3)
    th0 = workloads.theta0(w)
    th0 = (th0 + 0.02 * rng.standard_normal(th0.size)).astype(np.float32)
    ctx = gpu_ctx(w, theta0=th0)
    orc = oracle_run(w, theta0=th0)
    ctx.local_step()
    g = ctx.grads.cpu().numpy()
    loss = ctx.read_loss()
    for k in (0, dims["K"] - 1):
        want, wl = orc.grad(k, 0, th0.astype(np.float64))
        assert loss[k] == pytest.approx(wl, rel=1e-2)
        _assert_groups_close(w, g[k], want, "tiles k=%d" % k)
    ctx.close()


# Weight-gradient launches in every tile shape with ranges, of one block and of all blocks, and of each half of several blocks
# one after the other: the model, then what the plan makes of it, which the test holds it to.
PLANS = [
    (dict(d_in=192, d_hidden=1088, n_blocks=1, B_loc=3000, K=8), [("mlp", "192x384", 3)]),
    (dict(d_in=64, d_hidden=1088, n_blocks=1, B_loc=3000, K=8), [("mlp", "128x128", 3)]),
    (dict(d_in=128, d_hidden=576, n_blocks=1, B_loc=1500, K=8), [("mlp", "128x128 two groups", 3)]),
    (dict(d_in=64, d_hidden=64, n_blocks=2, B_loc=1040, K=1), [("all", "64x64 four groups", 3)]),
    (dict(d_in=320, d_hidden=320, n_blocks=2, B_loc=2050, K=8), [("all", "192x384", 4)]),
    (dict(d_in=64, n_heads=1, seq_len=41, d_hidden=64, n_blocks=2, B_loc=2050, K=1), [("all", "64x64 four groups", 4)]),
    (dict(d_in=128, n_heads=2, seq_len=41, d_hidden=64, n_blocks=2, B_loc=2050, K=7), [("all", "128x128 two groups", 3)]),
    (dict(d_in=192, n_heads=3, seq_len=50, d_hidden=192, n_blocks=2, B_loc=3000, K=6), [("all", "192x384", 4)]),
    (dict(d_in=64, d_hidden=576, n_blocks=2, B_loc=130, K=40), [("mlp", "128x128", 1)]),
    (dict(d_in=192, n_heads=3, seq_len=50, d_hidden=64, n_blocks=2, B_loc=5000, K=16),
     [("mlp", "64x64 four groups", 2), ("attention", "128x128 two groups", 1)]),
]


@pytest.mark.parametrize("dims,want", PLANS)
def test_gradient_by_weight_gradient_plan(dims, want):
    """Groups of a hundred thousand entries: one in 100 000 of the MLP's may pass the bound, as in test_gpu_parity.py."""
    heads = "n_heads" in dims
    model = (dims["K"], dims["B_loc"], dims["d_in"], dims["d_hidden"], dims["n_blocks"], int(heads))
    assert [p[1:4] for p in wgrad_host.plans([model])] == want
    w = workloads.get("vit" if heads else "resmlp", T=4, T_warm=1, **dims)
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
            _assert_groups_close(w, g[k], want_g, "plan k=%d" % k, tail=VIT_TAIL, weights_only_tail=True)
        else:
            _assert_groups_close(w, g[k], want_g, "plan k=%d" % k, tail=(1e-5, 1.5))
