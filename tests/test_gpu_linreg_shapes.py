"""GPU: the least-squares iteration in two kernels (up to 16 workers and 32 or 64 samples per wavefront; more beyond) at the sizes where it can go
wrong: feature counts that are no multiple of 4 or 64, few and many samples per wavefront, the largest number of
workers of a workgroup, workers that fit a workgroup and ones that do not; one by one and in one call (enqueued together or
replayed), against each other bit for bit and against the oracle."""
import numpy as np
import pytest

import workloads
from util import assert_mirror_matches_device, assert_params_close, gpu_ctx, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,d,B,opt", [(3, 1003, 17, "sgdm"), (16, 131, 76, "sgdm"), (17, 66, 9, "sgdm"), (1, 5, 1, "sgdm"),
                                       (5, 65, 33, "adamw"), (9, 1024, 8, "adamw"), (4, 64, 128, "sgdm"), (2, 3, 5, "adamw"),
                                       (9, 66, 32, "sgdm"), (9, 66, 33, "adamw"), (8, 70, 128, "sgdm"), (8, 70, 129, "sgdm"),
                                       # rows of 4 to 7 columns: both ends of a row in one or two groups
                                       (2, 4, 5, "sgdm"), (2, 6, 7, "sgdm"), (3, 7, 70, "sgdm"), (2, 1, 6, "sgdm"), (2, 2, 7, "sgdm"),
                                       # many samples of such rows
                                       (8, 6, 128, "sgdm"), (8, 67, 128, "sgdm"), (8, 3, 128, "sgdm"), (3, 4098, 5, "sgdm"), (3, 4097, 5, "sgdm"),
                                       # no workers of one workgroup, 1024 workgroups: 128-bit accesses inside short rows
                                       (17, 3, 64, "sgdm"), (17, 6, 64, "sgdm"), (17, 7, 64, "sgdm"),
                                       # ... and all workers in the gradient's workgroups: one wavefront each with 32 samples, three with
                                       # 34 and a shorter last run, eight with 64
                                       (16, 1100, 32, "sgdm"), (5, 1027, 100, "adamw"), (2, 1030, 500, "sgdm")])
def test_least_squares_shapes(K, d, B, opt):
    import torch
    kw = dict(mu=0.9, lam=1e-4) if opt == "sgdm" else dict(beta1=0.9, beta2=0.99, eps=1e-3, lam=0.01)
    w = workloads.get("lsq", K=K, d_in=d, B_loc=B, T=40, opt=opt, eta_max=0.1 / (1 + d / B), alpha=0.2 / (1 + d / B), **kw)
    orc = oracle_run(w)
    orc.step(40)
    ctx = gpu_ctx(w)
    ctx.step(40)
    with torch.cuda.stream(torch.cuda.Stream()):
        rep = gpu_ctx(w)
        rep.run(40)
        rep.stream.synchronize()
    for a, b in ((ctx.params, rep.params), (ctx.grads, rep.grads), (ctx.state0, rep.state0)):
        assert torch.equal(a, b)
    assert np.array_equal(ctx.read_loss(), rep.read_loss())
    p = ctx.params.cpu().numpy()
    assert list(ctx.read_sync_log()[0]) == list(orc.sync_log) and all(np.array_equal(p[k], p[0]) for k in range(K))
    assert_mirror_matches_device(rep)
    assert_params_close(p, orc.theta, what="params")
    ctx.close(); rep.close()
    # one gradient and loss by themselves
    ctx = gpu_ctx(w)
    ctx.local_step()
    g, loss = ctx.grads.cpu().numpy(), ctx.read_loss()
    for k in range(K):
        want, wl = orc.grad(k, 0, np.zeros(d))
        assert_params_close(g[k], want, what="grad k=%d" % k)
        assert loss[k] == pytest.approx(wl, rel=1e-5)
    ctx.close()


def test_more_samples_than_one_launch_takes():
    """One workgroup of 320 threads per sample, and at most 2^32 - 1 threads in a grid dimension: 13.4 M samples."""
    B = (1 << 32) // 320 + 2
    w = workloads.get("lsq", K=1, d_in=1, B_loc=B, T=2, eta_max=0.01, alpha=0.0)
    wstar = workloads.model_const(w).astype(np.float32)         # theta = w*: residuals of the noise alone, a sum that stays small
    X, y = oracle_run(w, theta0=wstar).linreg_batch(0, 0)
    ctx = gpu_ctx(w, theta0=wstar)
    ctx.local_step()
    ws = ctx.workspace.cpu().numpy().view(np.float32)
    x, r = ws[:B], ws[(B + 63) // 64 * 64:][:B]                # the two arrays of the workspace, 256-byte aligned
    want = X[:, 0] * wstar.astype(np.float64)[0] - y
    assert np.max(np.abs(x - X[:, 0])) < 2e-6                   # 5.4 at most, four ulps
    assert np.max(np.abs(r - want)) < 2e-6
    # an fp32 sum of B terms, one after the other: a random walk of B roundings of up to half an ulp of the partial sum
    terms = want * X[:, 0]
    walk = 2.0 ** -24 * np.max(np.abs(np.cumsum(terms))) * np.sqrt(B / 3)
    assert abs(ctx.grads.item() - np.mean(terms)) < 4 * walk / B
    assert ctx.read_loss()[0] == pytest.approx(0.5 * np.mean(want * want), rel=1e-4)
    ctx.close()


def test_more_features_than_one_fused_launch_takes():
    """2^28 features: 64 to a workgroup of 1024 threads would be 2^32 threads."""
    import torch
    import paper_2310_14423_amd as qsr
    d = (1 << 28) + 4
    w = workloads.get("lsq", K=1, d_in=d, B_loc=1, T=3, H_base=2, mu=0.9, lam=0.0, eta_max=0.25, alpha=0.0, data_sigma=0.0)
    ctx = qsr.Context(w, model_const=np.full(d, 2.0 ** -14, dtype=np.float32))      # theta = 0
    ctx.step(1)
    ws = ctx.workspace.view(torch.float32)
    x, r = ws[:d], ws[(d + 63) // 64 * 64]
    # a quarter of a thousand threads add up 2^20 products each, one after the other: 2^-24 sqrt(2^20 / 3) of the sum, times four
    assert float(r) == pytest.approx(-float(x.sum(dtype=torch.float64)) * 2.0 ** -14, rel=2e-4, abs=2e-4)
    assert torch.equal(ctx.grads[0], r * x) and torch.equal(ctx.state0, ctx.grads) and torch.equal(ctx.params, -0.25 * ctx.grads)
    assert ctx.read_loss()[0] == pytest.approx(0.5 * float(r) ** 2, rel=1e-6)
    assert ctx.get_state() == (1, 0, 1, 2)
    ctx.close()
