"""GPU: contexts on a stream other than the null stream, whose kernels do not wait for the null stream."""
import pytest

import workloads
from util import assert_mirror_matches_device, assert_params_close, gpu_ctx, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,kw", [
    ("lsq", dict(K=8, d_in=70, B_loc=128, T=60, eta_max=0.06, alpha=0.12)),      # iterations replayed from a graph
    ("flat60m", dict(K=4, P=1 << 18, T=60, eta_max=1e-3, alpha=0.004)),          # enqueued one by one
])
def test_context_made_while_the_null_stream_is_busy(name, kw):
    """Nothing that qsr_init does may be ordered behind work on the null stream and land on live state later."""
    import torch
    w = workloads.get(name, **kw)
    orc = oracle_run(w)
    orc.step(60)
    gpu_ctx(w).close()                            # library and allocator warm: making the next one is quick
    a = torch.ones(8192, 8192, device="cuda")
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)
    torch.cuda.synchronize()
    for _ in range(60):                           # 0.4 s or so
        torch.mm(a, a, out=b)
    busy = torch.cuda.Event()
    busy.record()
    with torch.cuda.stream(torch.cuda.Stream()):
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
