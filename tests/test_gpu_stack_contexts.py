"""rt_stack_prefill on several contexts of one process: calls of different contexts queued behind each other, on different streams and
from different threads give what one context alone gives - as launches per position (RT_FLAG_ENGINE_STEPWISE), whose calls take their side
streams from one pool, and on groups of workgroups."""
import threading

import pytest

from paper_2604_21215_amd import inputs as gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("form", ["launches", "groups"])
@pytest.mark.parametrize("threads", [False, True])
def test_contexts_share_side_streams(threads, form):
    from paper_2604_21215_amd import binding, torch_io as tio
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    B, N, d, L, n = 2, 150, 256, 4, 6   # more contexts at once than the pool keeps
    dls = [tio.DeviceLayer(gen.make_layer_weights(91, l, d, 4 * d, "bf16"), None, "bf16") for l in range(L)]
    x = tio.to_device(gen.make_custom(92, "bf16", B, N, d, 4, 4 * d).x, "bf16")
    ws = [dl.struct for dl in dls]
    torch.cuda.synchronize()

    def tensors():
        return ([torch.empty_like(x) for _ in range(L)], [torch.empty((N, B, 4, 64), dtype=x.dtype, device=x.device) for _ in range(L)],
                [torch.empty((N, B, 4, 64), dtype=x.dtype, device=x.device) for _ in range(L)])

    streams = [torch.cuda.Stream() for _ in range(n)]
    ctxs = [binding.RTContext(d, 4, 4 * d, B, N, "bf16", resid_scale=0.5, rms_eps=1e-6, reserve_stack_layers=L, stream=s.cuda_stream,
                              flags=binding.RT_FLAG_ENGINE_STEPWISE if form == "launches" else 0)
            for s in streams]
    outs = [tensors() for _ in range(n)]
    torch.cuda.synchronize()
    try:
        def go(k):
            for _ in range(2):
                ctxs[k].rt_stack_prefill(ws, x, *outs[k])

        if threads:
            pool = [threading.Thread(target=go, args=(k,)) for k in range(n)]
            for p in pool:
                p.start()
            for p in pool:
                p.join()
        else:
            for k in range(n):
                go(k)
        torch.cuda.synchronize()
        assert all(c.engine_form() == form and c.device_wait_expired() == 0 for c in ctxs)
        for k in range(1, n):
            for a, b in zip(outs[0], outs[k]):
                assert all(torch.equal(p, q) for p, q in zip(a, b))
        assert all(bool(torch.isfinite(t).all()) for t in outs[0][0])
    finally:
        for c in ctxs:
            c.rt_destroy()


@pytest.mark.parametrize("form", ["launches", "groups"])
def test_captured_call_replays(form):
    """a call recorded in a HIP graph: its replays read the tensors of the recorded call whatever ran on the context since, and give the
    eager call's bits on the inputs of the moment"""
    from paper_2604_21215_amd import binding, torch_io as tio
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    B, N, d, L = 2, 150, 256, 4
    sets = [[tio.DeviceLayer(gen.make_layer_weights(seed, l, d, 4 * d, "bf16"), None, "bf16") for l in range(L)] for seed in (93, 94)]
    xs = [tio.to_device(gen.make_custom(seed, "bf16", B, N, d, 4, 4 * d).x, "bf16") for seed in (95, 96, 97)]
    torch.cuda.synchronize()

    def tensors():
        return ([torch.zeros_like(xs[0]) for _ in range(L)], [torch.zeros((N, B, 4, 64), dtype=xs[0].dtype, device="cuda:0") for _ in range(L)],
                [torch.zeros((N, B, 4, 64), dtype=xs[0].dtype, device="cuda:0") for _ in range(L)])

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = binding.RTContext(d, 4, 4 * d, B, N, "bf16", resid_scale=0.5, rms_eps=1e-6, reserve_stack_layers=L, stream=stream.cuda_stream,
                                flags=binding.RT_FLAG_ENGINE_STEPWISE if form == "launches" else 0)
        try:
            refs = []
            for x in xs:
                refs.append(tensors())
                ctx.rt_stack_prefill([dl.struct for dl in sets[0]], x, *refs[-1])
            x, out, other = torch.empty_like(xs[0]), tensors(), tensors()
            stream.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                ctx.rt_stack_prefill([dl.struct for dl in sets[0]], x, *out)
            for x_new, ref in zip(xs, refs):
                ctx.rt_stack_prefill([dl.struct for dl in sets[1]], xs[2], *other)   # other descriptors on the same context
                x.copy_(x_new)
                graph.replay()
                stream.synchronize()
                assert all(torch.equal(p, q) for a, b in zip(out, ref) for p, q in zip(a, b))
            assert ctx.engine_form() == form and ctx.device_wait_expired() == 0
        finally:
            stream.synchronize()
            ctx.rt_destroy()


@pytest.mark.parametrize("L", [3, 6])
def test_phase_stamps_of_a_stack(monkeypatch, L):
    """rt_phase_trace after a stack on groups: a row per position of the last layer that the first group ran, not one per position of a chunk"""
    from paper_2604_21215_amd import binding, torch_io as tio
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    B, N, d = 2, 150, 256
    monkeypatch.setenv("RT_PERSIST_TRACE", "1")
    ctx = binding.RTContext(d, 4, 4 * d, B, N, "bf16", resid_scale=0.5, rms_eps=1e-6, reserve_stack_layers=L)
    try:
        dl = tio.DeviceLayer(gen.make_layer_weights(98, 0, d, 4 * d, "bf16"), None, "bf16")
        x = tio.to_device(gen.make_custom(99, "bf16", B, N, d, 4, 4 * d).x, "bf16")
        y, K, V = ([torch.zeros(s, dtype=x.dtype, device=x.device) for _ in range(L)] for s in ((B, N, d), (N, B, 4, 64), (N, B, 4, 64)))
        torch.cuda.synchronize()
        ctx.rt_stack_prefill([dl.struct] * L, x, y, K, V)
        torch.cuda.synchronize()
        assert ctx.engine_form() == "groups"
        rows = ctx.phase_trace(N).astype("int64").reshape(-1)
        assert rows.size == 16 * N and rows[0] > 0 and (rows[1:] >= rows[:-1]).all()
    finally:
        ctx.rt_destroy()
