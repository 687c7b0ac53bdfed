"""GPU: the block models' gradients at the sizes where the GEMMs change their tile shape or split, against the
oracle with the bf16 tolerances of test_gpu_parity.py (which also says where they come from)."""
import numpy as np
import pytest

import workloads
from test_gpu_parity import _assert_groups_close
from util import gpu_ctx, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [
    # NT GEMMs with N = d_hidden on 128 x 128 tiles (192 of them, ragged rows), N = d_in on 64 x 64, two stages
    dict(d_in=64, d_hidden=1024, n_blocks=1, B_loc=700, K=4),
    # on 128 x 256 tiles (1024 of them: the first number that takes them), the last row tile ragged
    dict(d_in=64, d_hidden=4096, n_blocks=1, B_loc=1021, K=8),
    # N = 192: one and a half 128 x 128 tiles wide
    dict(d_in=192, d_hidden=64, n_blocks=1, B_loc=4000, K=8),
    # weight gradients on 128 x 128 tiles with two groups (128 of them), a short token count for both groups
    dict(d_in=64, d_hidden=2048, n_blocks=1, B_loc=300, K=8),
    # reductions long enough to be cut into ranges: on 128 x 128 tiles, the last range ragged
    dict(d_in=64, d_hidden=128, n_blocks=1, B_loc=4129, K=2),
    # on 192 x 384 tiles (48 of them, rows and columns beyond the matrix)
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
