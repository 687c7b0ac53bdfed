"""GPU: contexts on a stream other than the null stream, whose kernels do not wait for the null stream and whose
iterations a caller may record into a graph of their own."""
import pytest

import workloads
from util import assert_mirror_matches_device, assert_params_close, gpu_ctx, oracle_run

pytestmark = pytest.mark.gpu


def _stream_beside_null():
    """A stream whose kernels run while the null stream is busy (there are only a few hardware queues, and a stream may share
    the null stream's)."""
    import time
    import torch
    x = torch.zeros(16, device="cuda")
    a = torch.ones(8192, 8192, device="cuda")
    torch.mm(a, a)
    torch.cuda.synchronize()
    for _ in range(30):                           # on the null stream, 0.2 s or so
        torch.mm(a, a)
    null = torch.cuda.Event()
    null.record()
    found = None
    for _ in range(16):
        s, done = torch.cuda.Stream(), torch.cuda.Event()
        with torch.cuda.stream(s):
            x.add_(1.0)
            done.record()
        time.sleep(0.003)
        if done.query() and not null.query():
            found = s
            break
    torch.cuda.synchronize()
    assert found is not None
    return found


@pytest.mark.parametrize("name,kw", [
    ("lsq", dict(K=8, d_in=70, B_loc=128, T=60, eta_max=0.06, alpha=0.12)),      # iterations enqueued together
    ("lsq", dict(K=5, d_in=1100, B_loc=24, T=60, eta_max=0.002, alpha=0.004)),   # iterations replayed from a graph
    ("flat60m", dict(K=4, P=1 << 18, T=60, eta_max=1e-3, alpha=0.004)),          # enqueued one by one
])
def test_context_made_while_the_null_stream_is_busy(name, kw):
    """Nothing that qsr_init does may be ordered behind work on the null stream and land on live state later."""
    import torch
    w = workloads.get(name, **kw)
    orc = oracle_run(w)
    orc.step(60)
    gpu_ctx(w).close()                            # library and allocator warm: making the next one is quick
    side = _stream_beside_null()
    a = torch.ones(8192, 8192, device="cuda")
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)
    torch.cuda.synchronize()
    for _ in range(60):                           # 0.4 s or so
        torch.mm(a, a, out=b)
    busy = torch.cuda.Event()
    busy.record()
    with torch.cuda.stream(side):
        ctx = gpu_ctx(w)
        ctx.run(20)
        ctx.stream.synchronize()
        assert not busy.query(), "the null stream was through before the context's first steps"
        assert ctx.get_state()[0] == 20
        busy.synchronize()                        # what waited for the null stream would have run by now
        ctx.run(40)
        assert list(ctx.read_sync_log()[0]) == list(orc.sync_log)
        assert ctx.get_state() == (60, len(orc.sync_log), 0, 0)
        assert_mirror_matches_device(ctx)
        assert_params_close(ctx.params.cpu().numpy(), orc.theta, what=name)
        ctx.close()


@pytest.mark.parametrize("name,kw", [
    ("lsq", dict(K=3, d_in=66, B_loc=9, eta_max=0.02, alpha=0.0)),
    ("lsq", dict(K=17, d_in=66, B_loc=9, eta_max=0.02, alpha=0.0)),
    ("mlp", dict(d_in=72, d_hidden=96, d_out=10, B_loc=48, K=3, milestones=(60, 100), eta_max=0.02, alpha=0.0)),
    ("flat60m", dict(K=3, P=9001, alpha=0.0, clip_norm=0.05)),
    ("flat60m", dict(K=3, P=9001, alpha=0.0, fuse_sync=True)),
    ("flat60m", dict(K=4, P=1 << 18, alpha=0.0, parallel=True)),
])
def test_iteration_recorded_by_the_caller(name, kw):
    """One iteration (every one ends a round) in the caller's graph: each replay counts and continues."""
    import torch
    w = workloads.get(name, T=150, H_base=1, power=0, **kw)
    ref = gpu_ctx(w)
    ref.step(13)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ctx = gpu_ctx(w)
        ctx.step(3)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            ctx.step(1)
        for done, replays in ((5, 2), (8, 3), (13, 5)):
            for _ in range(replays):
                graph.replay()
            assert ctx.get_state() == (done, done, 0, 1)
        assert list(ctx.read_sync_log()[0]) == list(range(1, 14))
        side.synchronize()
    for a, b in ((ctx.params, ref.params), (ctx.state0, ref.state0), (ctx.grads, ref.grads)):
        assert torch.equal(a, b)
    ctx.close(); ref.close()


def test_replays_are_held_against_the_mirror():
    """Recorded launches make no check of their own: a device that has gone another way than the host's mirror (here
    one step ahead, by a graph of the caller's) is reported by the next call that reads the state."""
    import torch
    import paper_2310_14423_amd as qsr
    w = workloads.get("flat60m", K=2, P=1024, T=150, H_base=3, power=0, alpha=0.0)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ctx = gpu_ctx(w)
        ctx.run(39)
        assert ctx.get_state() == (39, 13, 0, 3)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            ctx.step(1)
        graph.replay()
        assert ctx.get_state() == (40, 13, 1, 3)        # recorded once, run once
        graph.replay()                                  # ends no round either, as recorded
        with pytest.raises(qsr.QSRError) as e:
            ctx.get_state()
        assert e.value.code == -6
        ctx.restart()
        ctx.run(40)
        assert ctx.get_state() == (40, 13, 1, 3)
        ctx.close()
