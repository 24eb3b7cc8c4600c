"""rt_layer_prefill and rt_decode_step recorded in a HIP graph, in each form: replays on new inputs, with eager calls of the same context in between, give the
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


@pytest.mark.parametrize("B,d,form", [(2, 256, "one-launch"), (8, 1024, "one-launch"), (20, 256, "one-launch"), (60, 256, "launches")])
def test_replays_of_decoding_steps(B, d, form):
    """two steps of two layers in one graph, each over a cache of its own"""
    from paper_2604_21215_amd import binding, torch_io as tio
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    H, t = d // 64, 70
    dls = [tio.DeviceLayer(gen.make_layer_weights(66, l, d, 4 * d, "bf16"), None, "bf16") for l in range(2)]
    xs = [tio.to_device(gen.make_custom(seed, "bf16", B, t + 1, d, H, 4 * d).x, "bf16") for seed in (67, 68, 69)]
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        ctx = binding.RTContext(d, H, 4 * d, B, t + 1, "bf16", attn_scale=0.125, rms_eps=1e-6, stream=stream.cuda_stream)
        try:
            caches = [[x.reshape(t + 1, B, H, 64).clone() for _ in range(4)] for x in xs]   # any rows serve as a cache
            rows = [x[:, 0].contiguous() for x in xs]

            def step(x_t, y, c):
                ctx.rt_decode_step(dls[0].struct, x_t, t, y[0], c[0], c[1])
                ctx.rt_decode_step(dls[1].struct, y[0], t, y[1], c[2], c[3])

            refs = []
            for x_t, c in zip(rows, caches):
                y = torch.empty((2, B, d), dtype=x_t.dtype, device=x_t.device)
                step(x_t, y, c)
                refs.append([y] + [k[t].clone() for k in c])
            x_t, y, c = torch.empty_like(rows[0]), torch.zeros_like(refs[0][0]), [torch.empty_like(k) for k in caches[0]]
            other = torch.empty_like(y)
            stream.synchronize()
            assert ctx.engine_form() == form
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                step(x_t, y, c)
            for k in (0, 1, 2, 1, 0):
                if k % 2:
                    step(rows[2], other, [v.clone() for v in caches[2]])
                x_t.copy_(rows[k])
                for dst, src in zip(c, caches[k]):
                    dst.copy_(src)
                    dst[t].zero_()
                graph.replay()
                stream.synchronize()
                assert all(torch.equal(p, q) for p, q in zip([y] + [v[t] for v in c], refs[k])), k
            assert ctx.device_wait_expired() == 0
        finally:
            stream.synchronize()
            ctx.rt_destroy()
