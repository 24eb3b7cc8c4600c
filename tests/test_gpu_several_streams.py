"""Calls whose workgroups wait for one another (a prompt through a stack, decoding steps, a backward pass, an fp32 and a bf16 prefill), from
one thread and one stream each, at the same time: every one gives the bits that it gives alone, and no wait expires."""
import threading

import pytest

from paper_2604_21215_amd import inputs as gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _job(kind, stream):
    from paper_2604_21215_amd import binding, torch_io as tio
    dtype = "f32" if kind == "f32" else "bf16"
    B, N, d, L = 2, 200, 256, 3 if kind == "stack" else 1
    H, td = d // 64, tio.torch_dtype(dtype)
    ctx = binding.RTContext(d, H, 4 * d, B, N, dtype, resid_scale=0.5, attn_scale=0.125, rms_eps=1e-6, stream=stream.cuda_stream,
                            reserve_stack_layers=L if kind == "stack" else 0,
                            reserve=binding.RT_RESERVE_BACKWARD if kind == "backward" else 0)
    dls = [tio.DeviceLayer(gen.make_layer_weights(31, l, d, 4 * d, dtype), None, dtype) for l in range(L)]
    x = tio.to_device(gen.make_custom(32, dtype, B, N, d, H, 4 * d).x, dtype)
    new = lambda *s, t=td: torch.zeros(s, dtype=t, device=x.device)  # noqa: E731
    y, K, V = [new(B, N, d) for _ in range(L)], [new(N, B, H, 64) for _ in range(L)], [new(N, B, H, 64) for _ in range(L)]
    rows = [x[:, t].contiguous() for t in range(40)]
    dx, grads = new(B, N, d, t=torch.float32), {k: new(*w.shape, t=torch.float32) for k, w in dls[0].t.items()}
    out = {"stack": y + K + V, "decode": y + K + V, "backward": [dx] + list(grads.values())}.get(kind, y + K + V)

    def run():
        if kind == "stack":
            ctx.rt_stack_prefill([dl.struct for dl in dls], x, y, K, V)
        elif kind == "decode":
            for t, x_t in enumerate(rows):
                ctx.rt_decode_step(dls[0].struct, x_t, t, y[0][0, :B], K[0], V[0])
        elif kind == "backward":
            ctx.rt_layer_backward(dls[0].struct, x, x, x, None, None, dx, grads)
        else:
            ctx.rt_layer_prefill(dls[0].struct, x, y[0], K[0], V[0])

    return ctx, run, out, (dls, x)   # the last: kept until the job is done


def test_waiting_calls_of_several_streams():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    kinds = ("stack", "decode", "backward", "f32", "bf16", "decode")
    jobs = [_job(kind, torch.cuda.default_stream() if kind == "bf16" else torch.cuda.Stream()) for kind in kinds]
    torch.cuda.synchronize()
    try:
        alone = []
        for _, run, out, _ in jobs:
            run()
            torch.cuda.synchronize()
            alone.append([t.clone() for t in out])
        torch.cuda.synchronize()

        def go(run):
            for _ in range(5):
                run()

        pool = [threading.Thread(target=go, args=(run,)) for _, run, _, _ in jobs]
        for p in pool:
            p.start()
        for p in pool:
            p.join()
        torch.cuda.synchronize()
        for kind, (ctx, _, out, _), ref in zip(kinds, jobs, alone):
            assert ctx.device_wait_expired() == 0, kind
            assert all(torch.equal(a, b) for a, b in zip(out, ref)), kind
            assert all(bool(torch.isfinite(t).all()) for t in out), kind
    finally:
        for ctx, _, _, _ in jobs:
            ctx.rt_destroy()
