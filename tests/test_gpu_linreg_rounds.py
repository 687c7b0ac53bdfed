"""GPU: least-squares rounds that end inside a launch of several iterations (csrc/grad_linreg.hip: the workers exchange their
parameters there, as many at a time as a workgroup has groups of wavefronts) give, bit for bit, what the same iterations give one by
one: worker counts around those groups for one to four wavefronts a row, rounds that end on a launch's first and last
iteration, several calls, a call that repeats iterations that the exchange still holds words of, a wait that is given up, and contexts on streams side by side."""
import ctypes as C

import numpy as np
import pytest

import paper_2310_14423_amd as qsr
import workloads
from util import assert_mirror_matches_device, gpu_ctx

pytestmark = pytest.mark.gpu


def same(a, b):
    import torch
    assert a.get_state() == b.get_state()
    for x, y in zip((a.params, a.grads, a.state0, a.state1), (b.params, b.grads, b.state0, b.state1)):
        assert x is y is None or torch.equal(x, y)
    assert np.array_equal(a.read_loss(), b.read_loss())


@pytest.mark.parametrize("K,d,B,opt", [
    (1, 1024, 32, "sgdm"), (4, 1021, 32, "sgdm"), (5, 1024, 9, "adamw"), (8, 1000, 20, "sgdm"), (9, 770, 5, "sgdm"),
    (5, 700, 25, "sgdm"), (6, 768, 25, "adamw"), (11, 513, 10, "sgdm"), (8, 512, 30, "sgdm"), (9, 260, 30, "adamw"),
    (16, 256, 32, "sgdm"), (16, 7, 3, "adamw")])
@pytest.mark.parametrize("H", [1, 3, 8, 11, 16])
def test_rounds_inside_launches(K, d, B, opt, H):
    kw = dict(mu=0.9, lam=1e-4) if opt == "sgdm" else dict(beta1=0.9, beta2=0.99, eps=1e-3, lam=0.01)
    w = workloads.get("lsq", K=K, d_in=d, B_loc=B, T=200, opt=opt, eta_max=0.1 / (1 + d / B), H_base=H, alpha=0.0, power=0, **kw)
    ref, ctx = gpu_ctx(w), gpu_ctx(w)
    for n in (3, 150, 47):
        ref.step(n)
        ctx.run(n)
        same(ref, ctx)
    assert_mirror_matches_device(ctx)
    assert list(ctx.read_sync_log()[1]) == list(ref.read_sync_log()[1])
    ctx.close(); ref.close()


@pytest.mark.parametrize("back", [2, 4, 6])
def test_iterations_repeated(back):
    """The schedule set back between calls, to where the next rounds end with iterations that the exchange still holds words of: the last
    launch of the first call leaves those of iterations 70 and 68, one in each set of words.  The second call's first round reads the first set
    and waits for iteration 70, 68 or 66, its second round the other one and waits for 72, 70 or 68: whichever set holds which, a word taken for
    new meets its reader in two of the three, with parameters that have moved since."""
    w = workloads.get("lsq", K=7, d_in=300, B_loc=20, T=90, H_base=2, alpha=0.0, power=0)
    ref, ctx = gpu_ctx(w), gpu_ctx(w)
    for c, go in ((ref, ref.step), (ctx, ctx.run)):
        go(70)
        c.set_state((70 - back, 35 - back // 2, 0, 2))
        go(20)
    same(ref, ctx)
    ctx.close(); ref.close()


def test_wait_given_up():
    """A worker that finds no word in the looks it may take (here none) leaves NaN, and every reading of the state says so until a state is
    installed, by either call; then the results are the right ones again."""
    w = workloads.get("lsq", K=5, d_in=700, B_loc=25, T=60, H_base=3, alpha=0.0, power=0)
    ref, ctx = gpu_ctx(w), gpu_ctx(w)
    th0 = ctx.params.clone()
    limit = qsr.lib().qsr_debug_wait_limit
    for install in (ctx.restart, lambda: ctx.set_state((0, 0, 0, 3))):
        assert limit(ctx._ctx, 0) == 0
        ctx.run(20)
        ctx.run(10)                         # and another call behind it
        for read in (ctx.get_state, ctx.get_H, ctx.read_sync_log, ctx.read_timing):
            with pytest.raises(qsr.QSRError) as e:
                read()
            assert e.value.code == -8
        assert ctx.params.isnan().all()
        assert limit(ctx._ctx, 1 << 27) == 0
        ctx.params.copy_(th0); ctx.state0.zero_()
        install()
        assert ctx.get_state() == (0, 0, 0, 3)
    ref.step(30)
    ctx.run(30)
    same(ref, ctx)
    ctx.close(); ref.close()


def masked_stream(units):
    """A stream that may use the first `units` compute units, and what destroys it."""
    import torch
    torch.cuda.current_stream()
    hip = C.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))
    mask, handle = (C.c_uint32 * 8)(*[min(max(units - 32 * i, 0), 32) and (1 << min(units - 32 * i, 32)) - 1 for i in range(8)]), C.c_void_p()
    assert hip.hipExtStreamCreateWithCUMask(C.byref(handle), C.c_uint32(8), mask) == 0
    return torch.cuda.ExternalStream(handle.value), lambda: hip.hipStreamDestroy(handle)


@pytest.mark.parametrize("K,d,B,H", [(8, 1000, 20, 1), (8, 256, 30, 3), (5, 700, 25, 7), (16, 300, 9, 40)])
def test_streams_with_few_compute_units(K, d, B, H):
    """64 compute units, fewer than 16 a worker: no worker waits for another there (none could: no look is allowed), the launches end with
    the rounds, and the results are the same."""
    import torch
    w = workloads.get("lsq", K=K, d_in=d, B_loc=B, T=150, eta_max=0.1 / (1 + d / B), H_base=H, alpha=0.0, power=0)
    ref = gpu_ctx(w)
    stream, destroy = masked_stream(64)
    with torch.cuda.stream(stream):
        ctx = gpu_ctx(w)
    torch.cuda.synchronize()
    assert qsr.lib().qsr_debug_wait_limit(ctx._ctx, 0) == 0
    for n in (2, 35, 113):
        ref.step(n)
        ctx.run(n)
        torch.cuda.synchronize()
        same(ref, ctx)
    assert_mirror_matches_device(ctx)
    ctx.close(); ref.close()
    destroy()


@pytest.mark.parametrize("where", ["null stream", "stream", "stream of 128 compute units"])
def test_where_workers_wait(where):
    """Elsewhere they do, but only for rounds that end before a launch does."""
    import torch
    w = workloads.get("lsq", K=8, d_in=500, B_loc=24, T=256, H_base=4, alpha=0.0, power=0)
    stream, destroy = masked_stream(128) if "128" in where else (torch.cuda.default_stream() if "null" in where else torch.cuda.Stream(), None)
    for H, waits in ((4, True), (16, False), (100, False)):
        ref = gpu_ctx(dict(w, H_base=H))
        with torch.cuda.stream(stream):
            ctx = gpu_ctx(dict(w, H_base=H))
        torch.cuda.synchronize()
        ref.step(64)
        qsr.lib().qsr_debug_wait_limit(ctx._ctx, 0)
        ctx.run(64)
        torch.cuda.synchronize()
        if waits:
            with pytest.raises(qsr.QSRError):
                ctx.get_state()
        else:
            same(ref, ctx)
        ctx.close(); ref.close()
    if destroy:
        destroy()


def test_side_by_side():
    """Contexts of sixteen workers on streams of their own, enqueued in turn: each one's launches wait only for their own workers."""
    import torch
    w = workloads.get("lsq", K=16, d_in=500, B_loc=24, T=240, H_base=1, alpha=0.0, power=0)
    ref = gpu_ctx(w)
    ref.step(240)
    ctxs = []
    for _ in range(4):
        with torch.cuda.stream(torch.cuda.Stream()):
            ctxs.append(gpu_ctx(w))
    torch.cuda.synchronize()
    for _ in range(4):
        for c in ctxs:
            c.run(60)
    torch.cuda.synchronize()
    for c in ctxs:
        same(ref, c)
        c.close()
    ref.close()
