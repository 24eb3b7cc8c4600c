"""The flags of an fp32 context keep what they ask for where small layers run as one cooperative launch: RT_FLAG_NO_MFMA the plain-ALU
kernels."""
import pytest

from paper_2604_21215_amd import inputs as gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _prefill(flags):
    from paper_2604_21215_amd import binding, torch_io as tio
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    B, N, d = 2, 70, 256
    li = gen.make_custom(51, "f32", B, N, d, 4, 4 * d, gains="random")
    ctx = binding.RTContext(d, 4, 4 * d, B, N, "f32", attn_scale=0.125, rms_eps=1e-6, flags=flags)
    try:
        out = tio.prefill(ctx, tio.DeviceLayer(li.weights, li.gains, "f32"), tio.to_device(li.x, "f32"))
        torch.cuda.synchronize()
        assert ctx.device_wait_expired() == 0
        return out
    finally:
        ctx.rt_destroy()


def test_no_mfma_runs_the_plain_alu_kernels():
    from paper_2604_21215_amd import binding as b
    plain = _prefill(b.RT_FLAG_NO_MFMA | b.RT_FLAG_ENGINE_STEPWISE)
    assert all(torch.equal(p, q) for p, q in zip(_prefill(b.RT_FLAG_NO_MFMA), plain))   # the sums of the same kernels
    assert not all(torch.equal(p, q) for p, q in zip(_prefill(0), plain))               # which the matrix cores' are not
