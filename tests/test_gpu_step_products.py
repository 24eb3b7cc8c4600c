"""The products of one position of many sequences (position-batched prefill): row tiles of 64 and 128 with ragged ends, the
shortest contraction (one k-tile, fewer than the ring holds), widths that are odd multiples of 128, both tile forms of W1, the
options of the epilogues; matrices that are not aligned to 16 bytes take the kernels that load into registers."""
import pytest

from tests.test_gpu_parity import _run_case
from tests.test_gpu_tiled_products import _shifted

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("B,N,d,F,kw", [
    (129, 35, 128, 128, {}),                                   # one sequence more than two row tiles; one k-tile in every product
    (192, 40, 384, 640, dict(alibi=8.0)),                      # whole row tiles; 3 and 5 k-tiles of 128
    (770, 34, 128, 4096, {}),                                  # W1 on 128 x 128 tiles, ragged last one; fewer k-tiles than the ring holds
    (642, 33, 384, 4096, dict(alibi=8.0)),                     # the same with six k-tiles: the ring wraps
    (300, 33, 1024, 4096, dict(gains="unit")),
])
def test_position_batched(oracle, B, N, d, F, kw):
    _run_case(oracle, "bf16", B, N, d, d // 64, F, alpha=0.7, kv_cap=N + 1, n_decode=1, expect_engine="position-batched",
              **dict(dict(gains="random", scale=0.5), **kw))


def test_norm_free(oracle):
    """every normalisation the identity"""
    import numpy as np
    from paper_2604_21215_amd import binding, inputs as gen
    from tests.parity_util import TOL
    from tests.test_gpu_parallel import _check, _setup
    B, N, d, H, F = 140, 34, 256, 4, 512
    li = gen.make_custom(54, "bf16", B, N, d, H, F)
    x64 = li.x.astype(np.float64)
    f64 = lambda a: {k: v.astype(np.float64) for k, v in a.items()}  # noqa: E731
    ref = oracle.Layer(f64(li.weights), H, gains=f64(li.gains), norm_free=True, alpha=0.7, attn_scale=0.02, eps=1e-6).prefill(x64)
    ctx, tio, dl, xd, y, K, V = _setup(li, B, N, d, H, F, resid_scale=0.7, attn_scale=0.02, rms_eps=1e-6, flags=binding.RT_FLAG_NORM_FREE)
    try:
        ctx.rt_layer_prefill(dl.struct, xd, y, K, V)
        torch.cuda.synchronize()
        assert ctx.engine_name() == "position-batched"
        _check("norm-free B=%d" % B, x64, ref, (tio.to_host(y), tio.to_host(K), tio.to_host(V)), TOL["bf16"])
    finally:
        ctx.rt_destroy()


def test_matrices_that_are_not_aligned():
    from paper_2604_21215_amd import binding, inputs as gen, torch_io as tio
    B, N, d = 130, 40, 128
    li = gen.make_custom(53, "bf16", B, N, d, 2, 256)
    ctx = binding.RTContext(d, 2, 256, B, N, "bf16", resid_scale=0.7, attn_scale=0.5, rms_eps=1e-6,
                            stream=torch.cuda.current_stream().cuda_stream)
    x = tio.to_device(li.x, "bf16")
    w = {k: tio.to_device(v, "bf16") for k, v in li.weights.items()}
    g = {k: tio.to_device(v, "bf16") for k, v in li.gains.items()}
    out = []
    try:
        for ww in (w, {k: _shifted(v) for k, v in w.items()}):
            y = torch.empty_like(x)
            K = torch.empty((N, B, 2, 64), dtype=x.dtype, device=x.device)
            V = torch.empty_like(K)
            ctx.rt_layer_prefill(binding.make_weights(dict(ww, **g)), x, y, K, V)
            torch.cuda.synchronize()
            out.append((y, K, V))
        for a, b in zip(*out):   # two roundings to bf16 of other sums on the way
            assert float((a.float() - b.float()).norm() / a.float().norm()) <= 2 * 2.0 ** -8
    finally:
        ctx.rt_destroy()
