"""A device-side wait that expires in one launch of a call that makes several: the report stands to the end of the call.  The limit of
one poll applies to the first launch alone, so that the launches behind it run through."""
import pytest

from paper_2604_21215_amd import inputs as gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _context(monkeypatch, limit, *args, **kw):
    from paper_2604_21215_amd import binding
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    if limit:
        monkeypatch.setenv("RT_SPIN_LIMIT", limit)
    ctx = binding.RTContext(*args, **kw)
    monkeypatch.delenv("RT_SPIN_LIMIT", raising=False)
    return ctx


@pytest.mark.parametrize("limit,expired", [("1:1", 1), (None, 0)])
def test_stack(monkeypatch, limit, expired):
    from paper_2604_21215_amd import torch_io as tio
    B, N, d, L = 2, 150, 256, 3
    ctx = _context(monkeypatch, limit, d, 4, 4 * d, B, N, "bf16", reserve_stack_layers=L)
    try:
        dl = tio.DeviceLayer(gen.make_layer_weights(5, 0, d, 4 * d, "bf16"), None, "bf16")
        x = tio.to_device(gen.make_custom(6, "bf16", B, N, d, 4, 4 * d).x, "bf16")
        y, K, V = ([torch.zeros(s, dtype=x.dtype, device=x.device) for _ in range(L)] for s in ((B, N, d), (N, B, 4, 64), (N, B, 4, 64)))
        torch.cuda.synchronize()
        ctx.rt_stack_prefill([dl.struct] * L, x, y, K, V)
        torch.cuda.synchronize()
        assert ctx.device_wait_expired() == expired
    finally:
        ctx.rt_destroy()


@pytest.mark.parametrize("limit,expired", [("1:1", 1), (None, 0)])
@pytest.mark.parametrize("p_min", [32, 64])
def test_chunks_of_rows(monkeypatch, limit, expired, p_min):
    """17 sequences: two launches, on groups of workgroups and (p_min 64) on all of them"""
    from paper_2604_21215_amd import torch_io as tio
    B, N, d = 17, 70, 256
    ctx = _context(monkeypatch, limit, d, 4, 4 * d, B, N, "bf16", p_min=p_min)
    try:
        dl = tio.DeviceLayer(gen.make_layer_weights(7, 0, d, 4 * d, "bf16"), None, "bf16")
        x = tio.to_device(gen.make_custom(8, "bf16", B, N, d, 4, 4 * d).x, "bf16")
        tio.prefill(ctx, dl, x)
        torch.cuda.synchronize()
        assert ctx.engine_name() == "persistent"
        assert ctx.device_wait_expired() == expired
    finally:
        ctx.rt_destroy()
