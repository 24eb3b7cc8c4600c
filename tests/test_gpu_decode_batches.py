"""Multi-launch decoding steps: products of more workgroups than compute units (two share one, one group of steps requested
ahead), with two, three and four 32-index steps per wavefront; and the attention over the cache where the number of
(sequence, head) pairs is no multiple of the four of a workgroup, over one split of 64 keys and over two."""
import pytest

from tests.test_gpu_parity import _run_case

pytestmark = pytest.mark.gpu


# workgroups of 64 outputs x 32 sequences: [Wq; Wk; Wv] 3 d, W1 F, [Wk; Wv] 2 d wide
@pytest.mark.parametrize("B,N,d,F", [(353, 6, 512, 1536), (225, 6, 768, 1024), (257, 5, 1024, 2048)])
def test_more_workgroups_than_compute_units(oracle, B, N, d, F):
    assert 3 * d // 64 * -(-B // 32) > 256
    _run_case(oracle, "bf16", B, N, d, d // 64, F, gains="random", scale=0.5, kv_cap=N, n_decode=2)


@pytest.mark.parametrize("B,N,d,H", [(35, 70, 192, 3), (33, 40, 64, 1), (50, 131, 192, 3)])
def test_heads_no_multiple_of_four(oracle, B, N, d, H):
    assert B * H % 4
    _run_case(oracle, "bf16", B, N, d, H, 4 * d, gains="random", scale=0.5, kv_cap=N, n_decode=3, alibi=8.0)
