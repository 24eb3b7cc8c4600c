"""rt_layer_prefill recorded in a HIP graph, in each form: replays on new inputs, with eager calls of the same context in between, give the
eager call's bits.  (Workgroups know each other's words by a number of the call; a replay must not take those of the replay before it.)"""
import pytest

from paper_2604_21215_amd import inputs as gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype,B,N,d,p_min,form", [
    ("bf16", 2, 70, 256, 0, "groups"), ("bf16", 17, 40, 256, 0, "groups"), ("bf16", 2, 2, 1024, 0, "one-launch"), ("bf16", 3, 150, 256, 64, "one-launch"),
    ("f32", 2, 70, 256, 0, "groups"), ("f32", 2, 70, 256, 16, "launches")])
def test_replays(dtype, B, N, d, p_min, form):
    from paper_2604_21215_amd import binding, torch_io as tio
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    H = d // 64
    dls = [tio.DeviceLayer(gen.make_layer_weights(seed, 0, d, 4 * d, dtype), None, dtype) for seed in (61, 62)]
    xs = [tio.to_device(gen.make_custom(seed, dtype, B, N, d, H, 4 * d).x, dtype) for seed in (63, 64, 65)]
    torch.cuda.synchronize()
    new = lambda: [torch.zeros(s, dtype=xs[0].dtype, device=xs[0].device) for s in ((B, N, d), (N, B, H, 64), (N, B, H, 64))]  # noqa: E731
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = binding.RTContext(d, H, 4 * d, B, N, dtype, p_min=p_min, attn_scale=0.125, rms_eps=1e-6, stream=stream.cuda_stream)
        try:
            refs = []
            for x in xs:
                refs.append(new())
                ctx.rt_layer_prefill(dls[0].struct, x, *refs[-1])
            x, out, other = torch.empty_like(xs[0]), new(), new()
            stream.synchronize()
            assert ctx.engine_form() == form
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                ctx.rt_layer_prefill(dls[0].struct, x, *out)
            for k, (x_new, ref) in enumerate(zip(xs + xs[::-1], refs + refs[::-1])):
                if k % 2:
                    ctx.rt_layer_prefill(dls[1].struct, xs[2], *other)
                x.copy_(x_new)
                graph.replay()
                stream.synchronize()
                assert all(torch.equal(p, q) for p, q in zip(out, ref)), k
            assert ctx.device_wait_expired() == 0
        finally:
            stream.synchronize()
            ctx.rt_destroy()
