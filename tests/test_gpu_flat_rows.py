"""GPU: rows of any length and alignment through the kernels that treat the [K][P] buffers as one vector or in
groups of four columns (averaging, clipped and fused updates, gradient fill), against the oracle; Parallel OPT's
update of a shared gradient row."""
import numpy as np
import pytest

import workloads
from test_gpu_parity import test_average_rows as average_rows_case
from test_gpu_parity import test_gradient_clipping as clipping_case
from util import assert_mirror_matches_device, assert_params_close, gpu_ctx, oracle_run

pytestmark = pytest.mark.gpu


# one, two and three columns beyond the last group of four; each kernel's largest K and the first beyond it, on either
# side of the sizes that take one or two columns per lane
@pytest.mark.parametrize("K,P", [(16, 257), (17, 258), (32, 1027), (33, 259), (64, 1030), (65, 515), (3, 2), (64, 4096),
                                 (7, 131073), (8, 131076), (17, 131076), (33, 131076), (16, 200001), (16, 375002), (17, 131074), (20, 2400003),
                                 (32, 1600001), (33, 1250003), (65, 330005),
                                 # aligned: 24e6 and 56e6 elements
                                 (12, 1999996), (12, 2000000), (20, 2800000), (20, 2800004), (33, 727272), (33, 727276),
                                 # not aligned: 6e6 and 24e6 elements, 200000 columns, 72e6, 100e6 and 150e6 elements
                                 (17, 352941), (31, 199997), (31, 200005), (33, 200005), (33, 200006), (65, 369231),
                                 (64, 1125001), (64, 1124997), (17, 5882355), (100, 1500001)])
def test_averaging_of_unaligned_rows(K, P):
    average_rows_case(K, P)


# rows shorter than, as long as and longer than the 512 elements a workgroup takes at a time
@pytest.mark.parametrize("opt", ["adamw", "sgdm"])
@pytest.mark.parametrize("K,P,extra", [(7, 3, {}), (6, 130, {}), (3, 511, {}), (5, 513, {}), (4, 1026, dict(fuse_sync=True)), (4, 1028, dict(fuse_sync=True)),
                                       # the fused synchronization's longest rows of one element per lane, and the first of four
                                       (3, 399999, dict(fuse_sync=True)), (3, 400001, dict(fuse_sync=True)),
                                       (5, 1001, dict(parallel=True, H_base=1, power=0, alpha=0.0)),
                                       (3, 400003, {}), (3, 400002, dict(parallel=True, H_base=1, power=0, alpha=0.0)),
                                       (3, 400004, dict(parallel=True, H_base=1, power=0, alpha=0.0))])
def test_clipped_updates_of_any_row_length(opt, K, P, extra):
    clipping_case(opt, K, P, extra)


@pytest.mark.parametrize("P", [20001, 20002, 20003])
def test_gradient_fill_of_unaligned_rows(P):
    """The separately filled gradient of rows that start off the 16-byte grid equals the aligned rows' draw."""
    w = workloads.get("flat60m", K=3, P=P, T=8)
    ctx = gpu_ctx(w)
    ref = gpu_ctx(dict(w, P=20004))
    ctx.local_step(); ref.local_step()
    assert np.array_equal(ctx.grads.cpu().numpy(), ref.grads.cpu().numpy()[:, :P])
    ctx.close(); ref.close()


@pytest.mark.parametrize("P", [1 << 18, (1 << 18) + 2, 4096])
def test_parallel_opt_state_between_the_calls(P):
    """Whether or not the update has closed the round already, the step counts after qsr_local_step and the round
    closes in qsr_maybe_sync; results and log follow the oracle."""
    w = workloads.get("flat60m", K=4, P=P, T=12, H_base=1, alpha=0.0, power=0, parallel=True, opt="sgdm", mu=0.9, eta_max=0.1)
    ctx, orc = gpu_ctx(w), oracle_run(w)
    for t in range(1, 12):
        ctx.local_step()
        assert ctx.get_state() == (t, t - 1, 1, 1)
        assert len(ctx.read_sync_log()[0]) == t - 1
        ctx.maybe_sync()
        assert ctx.get_state() == (t, t, 0, 1)
    ctx.step()
    assert ctx.get_state() == (12, 12, 0, 0)
    orc.step(12)
    assert_params_close(ctx.params.cpu().numpy(), orc.theta, what="parallel")
    assert list(ctx.read_sync_log()[0]) == list(orc.sync_log)
    assert_mirror_matches_device(ctx)
    ctx.close()


def test_averaging_of_very_large_buffers_in_a_run():
    """More than 5e8 elements of 9 to 16 workers, where the averaging of a run takes a kernel of its own: zero gradients
    and no decay leave the parameters to the averaging alone."""
    import torch
    K, P = 9, 55555560
    w = workloads.get("flat60m", K=K, P=P, T=4, opt="sgdm", mu=0.0, lam=0.0, eta_max=0.1, H_base=2, power=0, alpha=0.0, model="external")
    ctx = gpu_ctx(w)
    gen = torch.Generator(device="cuda").manual_seed(5)
    start = torch.randn(K, P, device="cuda", generator=gen)
    ctx.params.copy_(start)
    ctx.step(1)
    assert torch.equal(ctx.params, start)
    ctx.step(1)
    for c in range(0, P, 1 << 23):
        want = start[:, c:c + (1 << 23)].double().mean(0)
        got = ctx.params[:, c:c + (1 << 23)]
        assert bool((got == got[:1]).all())
        # the sum carries its rounding errors along: one rounding of it and one of the division
        assert bool(((got[0].double() - want).abs() <= 2.0 ** -23 * want.abs() + 1e-12).all())
    ctx.close()


@pytest.mark.parametrize("opt", ["adamw", "sgdm"])
@pytest.mark.parametrize("P", [3200001, 3200004])
def test_clipped_update_beyond_what_the_caches_hold(opt, P):
    """More than 16e6 elements take streaming accesses, fewer plain ones: the rows four workers have in common with five
    come out with the same bits."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(11)
    scale = torch.tensor([0.02, 1.9, 2.1, 60.0, 5.0], device="cuda")[:, None] / P ** 0.5
    start = torch.randn(5, P, device="cuda", generator=gen)
    grads = [torch.randn(5, P, device="cuda", generator=gen) * scale for _ in range(3)]
    ctxs = []
    for K in (4, 5):
        w = workloads.get("flat60m", K=K, P=P, T=50, opt=opt, mu=0.9, model="external", clip_norm=2.0, H_base=40, power=0, alpha=0.0)
        ctx = gpu_ctx(w)
        ctx.params.copy_(start[:K])
        for g in grads:
            ctx.grads.copy_(g[:K])
            ctx.step(1)
        ctxs.append(ctx)
    few, many = ctxs
    assert torch.equal(few.params, many.params[:4]) and torch.equal(few.state0, many.state0[:4])
    assert opt == "sgdm" or torch.equal(few.state1, many.state1[:4])
    assert not torch.equal(few.params, start[:4])
    few.close(); many.close()


@pytest.mark.parametrize("opt,lo,hi", [("adamw", 1499999, 1500000), ("adamw", 6000000, 6000001), ("sgdm", 1999999, 2000001), ("sgdm", 6999999, 7000002)])
def test_update_of_a_callers_gradient_where_its_accesses_change(opt, lo, hi):
    """One row on either side of the sizes that the update streams past the caches: the same entries, the same bits, and all rows
    of a longer buffer cut the same way."""
    import torch
    out = []
    for K, P in ((1, lo), (1, hi), (3, (hi + 2) // 3)):
        w = workloads.get("flat60m", K=K, P=P, T=40, opt=opt, model="external", mu=0.9, beta1=0.9, beta2=0.99, eps=1e-6, lam=0.01, H_base=9,
                          alpha=0.0, power=0)
        n = 3 * ((hi + 2) // 3)
        gen = torch.Generator(device="cuda").manual_seed(5)
        theta, g = torch.randn(n, generator=gen, device="cuda"), torch.randn(3, n, generator=gen, device="cuda")
        ctx = gpu_ctx(w, theta0=np.zeros(P, dtype=np.float32))
        flat = lambda x: x.reshape(-1)
        flat(ctx.params).copy_(theta[:K * P])
        for i in range(3):
            flat(ctx.grads).copy_(g[i][:K * P])
            ctx.step(1)
        out.append([flat(x).clone() for x in (ctx.params, ctx.state0) + ((ctx.state1,) if opt == "adamw" else ())])
        ctx.close()
    for other in out[1:]:
        assert all(torch.equal(a[:lo], b[:lo]) for a, b in zip(out[0], other))
    assert not torch.equal(out[0][0], theta[:lo])
