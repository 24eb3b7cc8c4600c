"""rt_layer_backward with more sequences than the single-launch reverse loop takes: the loop's products on the matrix cores from
three bf16 parts of their fp32 inputs, at the edges of their tiles (16 sequences, 16 or 32 outputs) and contraction pieces (64
indices over eight wavefronts: fewer pieces than wavefronts, whole groups, a ragged last group)."""
import numpy as np
import pytest

from paper_2604_21215_amd import inputs as gen
from tests.test_gpu_backward import _run

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# what stays is one rounding to bf16 (2^-9) of each operand of the batched products after the loop, as with fp32 products in it:
# four of them in a row
TOL = 4 * 2.0 ** -9


@pytest.mark.parametrize("B,N,d,F,kw", [
    (9, 40, 64, 64, {}),                                     # one piece of the contraction, four output tiles
    (16, 35, 192, 448, dict(alibi=8.0)),                     # a whole tile of sequences; 3, 6 and 7 pieces
    (17, 70, 320, 1280, {}),                                 # one sequence more than a tile; 5, 10 and 20 pieces
    (33, 34, 1024, 4096, dict(with_pair_grads=False)),       # 32 outputs per workgroup
    (2, 40, 1088, 1152, dict(scale=0.1)),                    # few sequences at a width the single launch does not take; 17, 34, 18 pieces
])
def test_backward_wide_batches(oracle, B, N, d, F, kw):
    _run(oracle, "bf16", B, N, d, d // 64, F, alpha=0.7, tol=TOL, **dict(dict(scale=0.25), **kw))


def _mlp_dx(B, N, d, F, seed, edit=None, grads=None):
    """dx where only the loop's products reach it: Wv = Wo = 0 (nothing through the attention), inputs of +-1 (RMS statistics of
    exactly 1), W1 of small multiples of 1/8 (pre-activations are exact sums).  Returns dx and the same from numpy in fp64."""
    from math import erf, pi, sqrt
    from paper_2604_21215_amd import binding, torch_io as tio
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    rng = np.random.default_rng(seed)
    r16 = lambda a: gen.round_to_bf16(np.asarray(a, dtype=np.float32))  # noqa: E731
    w = {k: r16(rng.standard_normal((d, d)) * 0.1) for k in ("Wq", "Wk")}
    w.update(Wv=np.zeros((d, d), np.float32), Wo=np.zeros((d, d), np.float32))
    w["W1"] = (rng.integers(1, 4, (F, d)) * rng.choice((-0.125, 0.125), (F, d))).astype(np.float32)
    w["W2"] = r16(rng.standard_normal((d, F)) * 0.5)
    x = rng.choice((-1.0, 1.0), (B, N, d)).astype(np.float32)
    z, gy = r16(rng.standard_normal((B, N, d))), r16(rng.standard_normal((B, N, d)))
    if edit:
        edit(w, x, gy)
    ctx = binding.RTContext(d, d // 64, F, B, N, "bf16", rms_eps=0.0, stream=torch.cuda.current_stream().cuda_stream)
    try:
        dl = tio.DeviceLayer(w, None, "bf16")
        dx = torch.empty((B, N, d), dtype=torch.float32, device="cuda:0")
        ctx.rt_layer_backward(dl.struct, tio.to_device(x, "bf16"), tio.to_device(z, "bf16"), tio.to_device(gy, "bf16"), None, None, dx, grads or {})
        torch.cuda.synchronize()
        got = dx.cpu().numpy().astype(np.float64)
    finally:
        ctx.rt_destroy()
    x64, g64, W1, W2 = x.astype(np.float64), gy.astype(np.float64), w["W1"].astype(np.float64), w["W2"].astype(np.float64)
    pre = x64 @ W1.T
    gelu_d = 0.5 * (1 + np.vectorize(erf)(pre / sqrt(2))) + pre * np.exp(-pre * pre / 2) / sqrt(2 * pi)
    return got, x64, g64, W1, W2, gelu_d


def test_loop_products_distance_from_fp64():
    """fp32 inputs, exact partial products, fp32 sums: two products of 256 and 8192 indices and the fp32 rounding of gelu' in between
    (one accumulator that rounds at every matrix instruction is off by 3.4e-7 of the norm in the second product alone)."""
    got, x, gy, W1, W2, gelu_d = _mlp_dx(9, 2, 256, 8192, 71)
    t = ((gy @ W2) * gelu_d) @ W1
    ref = gy + t - x * (x * t).mean(-1, keepdims=True)
    assert np.linalg.norm(got - ref) / np.linalg.norm(ref) <= 2.0 ** -22.25   # 2e-7


def test_loop_products_infinite_weight():
    """an infinite element of W2 gives signed infinities in the gradient of its unit's pre-activation, hence of its row of W1: the
    parts of a gradient below its head are zero here"""
    def edit(w, x, gy):
        w["W2"][3, 10] = np.inf
        w["W1"][10] *= 0.0625   # gelu' of that unit positive
        x[:] = x[0, 0]
        gy[..., 3] = -np.abs(gy[..., 3])
    gW1 = torch.empty((512, 256), dtype=torch.float32, device="cuda:0")
    _, x, gy, _, _, gelu_d = _mlp_dx(9, 1, 256, 512, 72, edit=edit, grads=dict(W1=gW1))
    assert (gelu_d[..., 10] > 1e-3).all() and (gy[..., 3] != 0).all()
    got = gW1.cpu().numpy()
    assert np.array_equal(got[10], -np.sign(x[0, 0]) * np.inf)
    assert np.isfinite(np.delete(got, 10, 0)).all()
