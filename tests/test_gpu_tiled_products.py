"""The products of 2048 rows and more, whose k-tiles are loaded straight into LDS: exact and ragged row tiles, the shortest
contraction, batch rows shorter than a row tile's 32 rows, and caller's tensors that are not aligned to 16 bytes (whose k-tiles are
staged through registers)."""
import numpy as np
import pytest

from paper_2604_21215_amd import inputs as gen
from tests.parity_util import TOL, oracle_layer
from tests.test_gpu_backward import _run
from tests.test_gpu_parallel import _check, _setup

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _shifted(t):
    """the same values four bytes into a buffer"""
    out = torch.empty(t.numel() + 2, dtype=t.dtype, device=t.device)[2:].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("B,N,d,F,shift", [(8, 256, 128, 128, False), (100, 21, 128, 256, False), (3, 683, 384, 1536, False),
                                           (8, 256, 128, 256, True)])
def test_recompute_many_rows(oracle, B, N, d, F, shift):
    H = d // 64
    li = gen.make_custom(51, "bf16", B, N, d, H, F, gains="unit" if shift else "random")
    x64 = li.x.astype(np.float64)
    lay = oracle_layer(oracle, li, H, alpha=0.7, attn_scale=0.5, eps=1e-6)
    ref = lay.prefill(x64)
    ctx, tio, dl, xd, y, K, V = _setup(li, B, N, d, H, F, resid_scale=0.7, attn_scale=0.5, rms_eps=1e-6)
    try:
        from paper_2604_21215_amd import binding
        zd = tio.to_device(gen.round_to_bf16(ref[0].astype(np.float32)), "bf16")
        struct = dl.struct
        if shift:
            xd, zd = _shifted(xd), _shifted(zd)
            w = {k: _shifted(tio.to_device(v, "bf16")) for k, v in li.weights.items()}
            w.update({k: tio.to_device(v, "bf16") for k, v in li.gains.items()})
            struct = binding.make_weights(w)
        ctx.rt_layer_recompute(struct, xd, zd, y, K, V)
        torch.cuda.synchronize()
        _check("recompute B=%d N=%d d=%d" % (B, N, d), x64, ref, (tio.to_host(y), tio.to_host(K), tio.to_host(V)), TOL["bf16"])
    finally:
        ctx.rt_destroy()


@pytest.mark.parametrize("gains,d", [("unit", 128), (None, 384)])
def test_tensors_that_are_not_aligned_give_the_same_bits(gains, d):
    """staged through registers the tiles are the same ones, summed in the same order"""
    from paper_2604_21215_amd import binding, torch_io as tio
    B, N, F = 5, 411, 256
    li = gen.make_custom(55, "bf16", B, N, d, d // 64, F)
    ctx, _, dl, xd, y, K, V = _setup(li, B, N, d, d // 64, F, resid_scale=0.7, attn_scale=0.5, rms_eps=1e-6)
    try:
        w = {k: tio.to_device(v, "bf16") for k, v in li.weights.items()}
        g = {k: tio.to_device(v, "bf16") for k, v in li.gains.items()} if gains else {}
        zd = tio.to_device(gen.round_to_bf16(np.random.default_rng(8).standard_normal((B, N, d)).astype(np.float32)), "bf16")
        outs = []
        for sh in (lambda t: t, _shifted):
            out = [torch.empty_like(t) for t in (y, K, V)]
            ctx.rt_layer_recompute(binding.make_weights(dict({k: sh(v) for k, v in w.items()}, **g)), sh(xd), sh(zd), *out)
            torch.cuda.synchronize()
            outs.append(out)
        assert all(torch.equal(a, b) for a, b in zip(*outs))
    finally:
        ctx.rt_destroy()


def test_backward_many_rows(oracle):
    _run(oracle, "bf16", 9, 57, 128, 2, 192, scale=0.25, alpha=0.7)


def test_backward_with_matrices_that_are_not_aligned(oracle):
    """the same gradients, bit for bit, from weights four bytes into their buffers"""
    from paper_2604_21215_amd import binding, torch_io as tio
    B, N, d, H, F = 9, 40, 128, 2, 256
    li = gen.make_custom(52, "bf16", B, N, d, H, F)
    ctx, _, dl, xd, y, K, V = _setup(li, B, N, d, H, F, rms_eps=1e-6)
    try:
        w = {k: tio.to_device(v, "bf16") for k, v in li.weights.items()}
        g = {k: tio.to_device(v, "bf16") for k, v in li.gains.items()}
        ctx.rt_layer_prefill(dl.struct, xd, y, K, V)
        got = []
        for ww in (w, {k: _shifted(v) for k, v in w.items()}):
            dx = torch.empty((B, N, d), dtype=torch.float32, device="cuda:0")
            grads = {k: torch.empty(v.shape, dtype=torch.float32, device="cuda:0") for k, v in w.items()}
            ctx.rt_layer_backward(binding.make_weights(dict(ww, **g)), xd, y, xd, None, None, dx, grads)
            torch.cuda.synchronize()
            got.append([dx] + [grads[k] for k in sorted(grads)])
        assert all(torch.equal(a, b) for a, b in zip(*got))
    finally:
        ctx.rt_destroy()
