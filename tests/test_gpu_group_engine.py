"""The sequential loop by groups of workgroups (p_min 32, up to 16 sequences): every number of sequences per group (1, 2, 4 rows
of the exchanged vectors, full and ragged), every width (odd multiples of 256 leave half a contraction chunk empty), lengths at
the edges of the direct window and of the blocks that stay in one workgroup (up to 512 keys) or are spread over a group."""
import pytest

from paper_2604_21215_amd import inputs as gen
from tests.test_gpu_backward import _run as _backward_case
from tests.test_gpu_parity import _run_case
from tests.test_gpu_stack import EMB_UNIT, _run_elementwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [256, 512, 768, 1024])
@pytest.mark.parametrize("B,N,alibi", [(1, 65, 0.0), (4, 34, 8.0), (5, 97, 0.0), (8, 33, 8.0), (9, 66, 0.0), (16, 64, 8.0)])
def test_rows_per_group(oracle, d, B, N, alibi):
    _run_case(oracle, "bf16", B, N, d, d // 64, 4 * d, gains="random", scale=0.5, alpha=0.7, alibi=alibi, kv_cap=N + 1,
              expect_engine="persistent")


@pytest.mark.parametrize("B,N,alibi", [(5, 1100, 0.0), (2, 1290, 8.0)])
def test_blocks_of_up_to_1024_keys(oracle, B, N, alibi):
    _run_case(oracle, "bf16", B, N, 256, 4, 1024, gains="random", scale=0.125, alibi=alibi, expect_engine="persistent")


@pytest.mark.parametrize("B,N,layers,d,alibi", [
    (1, 65, 1, 256, 0.0), (3, 64, 2, 512, 8.0), (4, 300, 5, 256, 0.0), (5, 129, 3, 768, 0.0), (8, 200, 4, 256, 8.0),
    (9, 130, 2, 256, 0.0), (16, 70, 6, 256, 8.0), (12, 70, 7, 256, 0.0)])
def test_stack(oracle, B, N, layers, d, alibi):
    """four, two or one layer at a time, more layers than run at once, chunks with a ragged last one, the first batch that leaves the
    engine again (nine sequences and more than six layers)"""
    wl = gen.Workload("stack_groups", "bf16", B, N, d, d // 64, 4 * d, layers=layers, vocab=300, decode_steps=2, seed=990 + B)
    _run_elementwise(oracle, wl, B, N, 2, emb_scale=EMB_UNIT, wavefront=True, alibi=alibi)


@pytest.mark.parametrize("B,N,d,alibi", [(1, 1, 128, 0.0), (2, 34, 256, 8.0), (3, 65, 384, 0.0), (8, 130, 128, 8.0), (9, 66, 256, 0.0),
                                         (16, 97, 384, 8.0), (4, 290, 256, 0.0), (1, 515, 128, 0.0), (32, 40, 128, 0.0)])
def test_fp32(oracle, B, N, d, alibi):
    """fp32 storage: one sequence per group and several, widths whose share of a contraction ends inside a chunk, blocks of 32 to 512 keys"""
    _run_case(oracle, "f32", B, N, d, d // 64, 4 * d, gains="random", scale=0.5, alpha=0.7, alibi=alibi, kv_cap=N + 1)


@pytest.mark.parametrize("d", [256, 512, 768, 1024])
@pytest.mark.parametrize("B,N,alibi", [(1, 33, 8.0), (4, 64, 0.0), (5, 70, 0.0), (8, 34, 8.0)])
def test_reverse_loop(oracle, d, B, N, alibi):
    """the backward pass's loop: one and two sequences per group, full and ragged, blocks of one position and whole ones"""
    _backward_case(oracle, "bf16", B, N, d, d // 64, 4 * d, alpha=0.7, scale=0.125, alibi=alibi, seed=77)


@pytest.mark.parametrize("B,N,d,alibi", [(130, 70, 256, 0.0), (129, 100, 320, 8.0)])
def test_merge_of_eight_lanes_per_row(oracle, B, N, d, alibi):
    """the position-batched merge: windows of 0 to 31 keys, none to two stored levels, heads that do not fill the last workgroup"""
    _run_case(oracle, "bf16", B, N, d, d // 64, 4 * d, gains="random", scale=0.5, alibi=alibi, expect_engine="position-batched")
