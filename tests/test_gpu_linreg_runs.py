"""GPU: least-squares iterations enqueued together (workers that fit one workgroup each: csrc/grad_linreg.hip) give, bit for
bit, what the same iterations give one by one, at the sizes where the kernel takes another form: one to four wavefronts a row,
two to eight samples a wavefront, padded rows, a wavefront left over, sixteen workers; rounds of one iteration, of several
launches and longer than the draws that are held; a call that ends inside a round and one that goes on from there."""
import numpy as np
import pytest

import workloads
from util import assert_mirror_matches_device, assert_params_close, gpu_ctx, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,d,B,H,opt", [
    (2, 256, 32, 1, "sgdm"), (3, 257, 16, 5, "adamw"), (1, 512, 64, 16, "sgdm"), (2, 513, 11, 17, "sgdm"), (2, 768, 40, 33, "adamw"),
    (2, 769, 32, 40, "sgdm"), (16, 1024, 32, 7, "sgdm"), (5, 1023, 31, 50, "sgdm"), (16, 3, 32, 9, "sgdm"), (1, 1, 1, 2, "sgdm"),
    (8, 61, 128, 36, "sgdm"), (2, 1022, 9, 16, "adamw")])
def test_together_and_one_by_one(K, d, B, H, opt):
    import torch
    kw = dict(mu=0.9, lam=1e-4) if opt == "sgdm" else dict(beta1=0.9, beta2=0.99, eps=1e-3, lam=0.01)
    T = 100
    w = workloads.get("lsq", K=K, d_in=d, B_loc=B, T=T, opt=opt, eta_max=0.1 / (1 + d / B), H_base=H, alpha=0.0, power=0, **kw)
    ref = gpu_ctx(w)
    states = []
    for n in (37, 2, 61):
        ref.step(n)
        states.append(([x.clone() for x in (ref.params, ref.grads, ref.state0) + ((ref.state1,) if opt == "adamw" else ())],
                       ref.read_loss(), ref.get_state()))
    ctx = gpu_ctx(w)                        # on the null stream too: nothing is recorded here
    for n, (want, loss, state) in zip((37, 2, 61), states):
        ctx.run(n)
        assert ctx.get_state() == state
        got = (ctx.params, ctx.grads, ctx.state0) + ((ctx.state1,) if opt == "adamw" else ())
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        assert np.array_equal(ctx.read_loss(), loss)
    assert_mirror_matches_device(ctx)
    orc = oracle_run(w)
    orc.step(T)
    assert list(ctx.read_sync_log()[0]) == list(orc.sync_log)
    # AdamW turns differences of an entry's smallest gradients into steps: the schedule above, and the parameters of SGD
    if opt == "sgdm":
        assert_params_close(ctx.params.cpu().numpy(), orc.theta, what="params")
    ctx.close(); ref.close()


def test_together_after_set_state():
    """The same, entered in the middle of a schedule."""
    import torch
    w = workloads.get("lsq", K=4, d_in=300, B_loc=20, T=120)
    a, b = gpu_ctx(w), gpu_ctx(w)
    a.step(50); b.step(50)
    for c in (a, b):
        c.set_state((20, 3, 0, 6))
    a.step(60)
    b.run(60)
    assert a.get_state() == b.get_state() and torch.equal(a.params, b.params) and torch.equal(a.state0, b.state0)
    a.close(); b.close()


@pytest.mark.parametrize("K,d,B,opt", [
    # rounds of one iteration in two kernels, samples shared out in the runs of the other kernel: one, two and five wavefronts a
    # worker, several runs a wavefront, a run cut short, workers without a second wavefront
    (4, 668, 25, "sgdm"), (16, 257, 8, "adamw"), (3, 1003, 17, "sgdm"), (2, 256, 32, "sgdm"), (1, 5, 3, "sgdm"), (11, 916, 17, "sgdm"),
    (6, 300, 16, "adamw"), (16, 1024, 32, "sgdm"), (8, 61, 128, "sgdm")])
def test_rounds_of_one_iteration(K, d, B, opt):
    """Long rounds, nineteen of one iteration, long ones, two of one iteration (fewer than are worth another way through the
    kernels), one to the end; entered and left at different places by the calls."""
    import torch
    kw = dict(mu=0.9, lam=1e-4) if opt == "sgdm" else dict(beta1=0.9, beta2=0.99, eps=1e-3, lam=0.01)
    T, eta = 100, 0.02 / (1 + d / B)
    w = workloads.get("lsq", K=K, d_in=d, B_loc=B, T=T, opt=opt, eta_max=7 * eta, H_base=1, alpha=7.5 * eta, power=1, **kw)
    table = np.full(T, eta)                                      # H = 7, but H = 1 where the rate is seven times as high
    table[21:40] = table[61:63] = 7 * eta
    for calls in ((100,), (23, 5, 33, 39), (2, 58, 40)):
        ref, ctx = gpu_ctx(w, eta_table=table), gpu_ctx(w, eta_table=table)
        for n in calls:
            ref.step(n)
            ctx.run(n)
            assert ctx.get_state() == ref.get_state()
            for a, b in zip((ctx.params, ctx.grads, ctx.state0, ctx.state1), (ref.params, ref.grads, ref.state0, ref.state1)):
                assert a is b is None or torch.equal(a, b)
            assert np.array_equal(ctx.read_loss(), ref.read_loss())
        H = list(ctx.read_sync_log()[1])
        assert H[:3] == [7] * 3 and H[3:22] == [1] * 19 and H[22:25] == [7] * 3 and H[25:27] == [1] * 2 and sum(H) == T
        assert_mirror_matches_device(ctx)
        ctx.close(); ref.close()
