"""rt_lm_head on the matrix cores at the edges of its tiles: vocabulary rows in tiles of 16 (remainders, rows that allow no
16-byte stores), batch tiles of up to 16 (fewer, full, one more; fewer rows where wide rows fill the LDS), row widths of one,
several and many blocks of 256, strided rows; and the plain-ALU form on both sides of the rule that takes it for few rows of both
kinds."""
import numpy as np
import pytest

from paper_2604_21215_amd import inputs as gen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d,vocab,B,norm_free", [(256, 1, 1, False), (256, 15, 16, False), (512, 4097, 17, False), (1024, 2064, 8, False),
                                                 (768, 33000, 5, False), (2048, 130, 33, False), (12288, 50, 3, False), (1024, 62, 9, True),
                                                 (1024, 2048, 5, False), (1024, 2048, 6, False), (512, 4096, 2, True), (512, 4097, 2, False),
                                                 (2048, 8192, 2, False)])
def test_lm_head_tiles(oracle, d, vocab, B, norm_free):
    from paper_2604_21215_amd import binding, torch_io as tio
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    rng = np.random.default_rng(d + vocab)
    W = gen.round_to_bf16((rng.standard_normal((vocab, d)) * 0.05).astype(np.float32))
    g = gen.round_to_bf16(rng.uniform(0.5, 1.5, d).astype(np.float32))
    z = gen.round_to_bf16(rng.standard_normal((B, 3, d)).astype(np.float32))
    ctx = binding.RTContext(d, d // 64, 4 * d, B, 8, "bf16", rms_eps=1e-6, flags=binding.RT_FLAG_NORM_FREE if norm_free else 0,
                            stream=torch.cuda.current_stream().cuda_stream)
    try:
        zd = tio.to_device(z, "bf16")
        out = torch.full((B + 1, vocab), float("nan"), dtype=torch.float32, device="cuda:0")   # one guard row behind
        ctx.rt_lm_head(tio.to_device(W, "bf16"), tio.to_device(g, "bf16"), zd[:, 1], zd.stride(0), B, out[:B])
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
    finally:
        ctx.rt_destroy()
    W64, z64, g64 = W.astype(np.float64), z[:, 1].astype(np.float64), g.astype(np.float64)
    ref = oracle.lm_head(W64, z64, g64, norm_free=True) if norm_free else oracle.lm_head(W64, z64, g64, eps=1e-6)
    n = z64 if norm_free else z64 / np.sqrt((z64 ** 2).mean(-1, keepdims=True) + 1e-6) * g64
    # fp32 operands and sums: rounding errors of 2^-24 of the partial sums, which grow like the root of the d terms; rows
    # rounded to bf16 would be off by 2^-9 / sqrt(3 d) of the sum of magnitudes, three times this bound at d = 1024
    bound = 8 * np.sqrt(d) * 2.0 ** -24 * (np.abs(n) @ np.abs(W64).T)
    assert np.all(np.abs(got[:B] - ref) <= bound)
    assert np.all(np.isnan(got[B]))


@pytest.mark.parametrize("d,vocab,B", [(256, 4096, 8), (512, 4096, 17), (1024, 4096, 8), (2048, 4096, 12)])
def test_lm_head_distance_from_fp64(d, vocab, B):
    """fp32 sums: the normalised rows carry up to 2^-24 of 1 / rms and two products' roundings (2^-24 / sqrt(3) of the norm each);
    the sums' own roundings add about as much.  2^-23 in all, where one accumulator per logit that rounds at every matrix
    instruction is off by 1.6e-7 (d = 256) to 4.8e-7 (d = 2048)."""
    from paper_2604_21215_amd import binding
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    g = torch.Generator(device="cuda:0")
    g.manual_seed(d)
    W = (torch.randn(vocab, d, generator=g, device="cuda:0") * 0.02).bfloat16()
    gain = (torch.randn(d, generator=g, device="cuda:0") * 0.1 + 1).bfloat16()
    z = torch.randn(B, d, generator=g, device="cuda:0").bfloat16()
    ctx = binding.RTContext(d, d // 64, 4 * d, B, 8, "bf16", rms_eps=1e-6, stream=torch.cuda.current_stream().cuda_stream)
    try:
        out = torch.empty((B, vocab), dtype=torch.float32, device="cuda:0")
        ctx.rt_lm_head(W, gain, z, d, B, out)
        torch.cuda.synchronize()
    finally:
        ctx.rt_destroy()
    z64 = z.double().cpu()
    ref = z64 / (z64.square().mean(-1, keepdim=True) + 1e-6).sqrt() * gain.double().cpu() @ W.double().cpu().T
    assert float((out.double().cpu() - ref).norm() / ref.norm()) <= 2.0 ** -23


@pytest.mark.parametrize("B", [2, 17])
def test_lm_head_infinite_weights(B):
    """one infinite weight in a row gives a signed infinity (the normalised values are cut into three parts, some of them zero or of
    the other sign), opposite ones or a zero value under one NaN; a normalised value beyond the largest bf16 stays finite"""
    from paper_2604_21215_amd import binding, torch_io as tio
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    d, vocab = 256, 30000
    rng = np.random.default_rng(5)
    z = np.zeros((B, d), np.float32)
    z[:, :254], z[:, 254] = rng.choice((-1.0, 1.0), (B, 254)), 0.5          # 1 / rms = 1.0034...
    g = np.ones(d, np.float32)
    g[7:20] = gen.round_to_bf16(rng.uniform(0.5, 1.5, 13).astype(np.float32))
    g[5] = np.float32(2.0 ** 128 - 2.0 ** 120)                              # the largest bf16
    W = gen.round_to_bf16((rng.standard_normal((vocab, d)) * 0.05).astype(np.float32))
    W[:, 5] = 0.0
    for v in range(256):                                                     # every place of an infinite weight
        W[v, v] = np.inf if v % 3 else -np.inf
    W[5, 5] = 2.0 ** -100
    W[300, 3], W[300, 90], W[301, 3], W[301, 90] = np.inf, -np.inf, np.inf, np.inf
    W[302, 5] = 0.125
    ctx = binding.RTContext(d, d // 64, 4 * d, B, 8, "bf16", rms_eps=1e-6, stream=torch.cuda.current_stream().cuda_stream)
    try:
        out = torch.empty((B, vocab), dtype=torch.float32, device="cuda:0")
        ctx.rt_lm_head(tio.to_device(W, "bf16"), tio.to_device(g, "bf16"), tio.to_device(z, "bf16"), d, B, out)
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
    finally:
        ctx.rt_destroy()
    z64 = z.astype(np.float64)
    n = z64 / np.sqrt((z64 ** 2).mean(-1, keepdims=True) + 1e-6) * g.astype(np.float64)
    assert 2.0 ** 128 - 2.0 ** 119 < np.abs(n).max() < 2.0 ** 128 - 2.0 ** 103   # fp32 holds it, rounding to bf16 does not
    with np.errstate(invalid="ignore", over="ignore"):
        ref = np.stack([(W.astype(np.float64) * n[b]).sum(-1) for b in range(B)])
    assert np.isinf(ref[:, :255]).sum() >= 254 * B and np.isnan(ref[:, 255]).all() and np.isfinite(ref[:, 303:]).all()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.where(np.isinf(got), np.sign(got), 0), np.where(np.isinf(ref), np.sign(ref), 0))
    ok = np.isfinite(ref)
    assert np.allclose(got[ok], ref[ok], rtol=1e-5, atol=1e-5)
