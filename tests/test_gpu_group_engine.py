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
              expect_engine="persistent", expect_form="groups")


@pytest.mark.parametrize("B,N,d,form", [(2, 1, 256, "one-launch"), (2, 2, 256, "groups"), (9, 2, 1024, "one-launch"), (1, 3, 1024, "groups")])
def test_first_positions(oracle, B, N, d, form):
    _run_case(oracle, "bf16", B, N, d, d // 64, 4 * d, gains="random", scale=0.5, alpha=0.7, expect_engine="persistent", expect_form=form)


@pytest.mark.parametrize("B,N,alibi", [(5, 1100, 0.0), (2, 1290, 8.0)])
def test_blocks_of_up_to_1024_keys(oracle, B, N, alibi):
    _run_case(oracle, "bf16", B, N, 256, 4, 1024, gains="random", scale=0.125, alibi=alibi, expect_engine="persistent",
              expect_form="groups")


@pytest.mark.parametrize("B,N,d,p_min", [(16, 140, 1024, 128), (8, 100, 1024, 64), (16, 70, 256, 64), (35, 70, 256, 64)])
def test_windows_that_keep_the_other_form(oracle, B, N, d, p_min):
    """a direct window of 64 keys and more: one launch of all 256 workgroups, with a (b, h) in each of them in the first case, and in
    chunks of sixteen sequences in the last"""
    _run_case(oracle, "bf16", B, N, d, d // 64, 4 * d, p_min=p_min, gains="random", scale=0.5, alpha=0.7, expect_engine="persistent",
              expect_form="one-launch")


@pytest.mark.parametrize("B,N,layers,d,alibi", [
    (1, 65, 1, 256, 0.0), (3, 64, 2, 512, 8.0), (4, 300, 5, 256, 0.0), (5, 129, 3, 768, 0.0), (8, 200, 4, 256, 8.0),
    (9, 130, 2, 256, 0.0), (16, 2, 1, 256, 0.0), (1, 3, 1, 256, 8.0), (3, 1, 5, 256, 0.0), (16, 70, 6, 256, 8.0), (12, 70, 7, 256, 0.0)])
def test_stack(oracle, B, N, layers, d, alibi):
    """four, two or one layer at a time, more layers than run at once, chunks with a ragged last one"""
    wl = gen.Workload("stack_groups", "bf16", B, N, d, d // 64, 4 * d, layers=layers, vocab=300, decode_steps=2, seed=990 + B)
    _run_elementwise(oracle, wl, B, N, 2, emb_scale=EMB_UNIT, wavefront=True, alibi=alibi, expect_form="groups")


@pytest.mark.parametrize("chunk", [128, 256])
@pytest.mark.parametrize("B,N,layers,alibi,poison", [(1, 515, 1, 8.0, False), (2, 300, 5, 0.0, True), (5, 391, 2, 8.0, False), (9, 290, 3, 8.0, True)])
def test_stack_with_longer_chunks(oracle, monkeypatch, chunk, B, N, layers, alibi, poison):
    """the chunks that long stacks take: blocks of 64 and 128 keys inside a chunk, the far tile for more than 128 queries, a ragged last
    chunk; four layers at a time, two and one"""
    monkeypatch.setenv("RT_GROUP_CHUNK", str(chunk))
    wl = gen.Workload("stack_chunks", "bf16", B, N, 256, 4, 1024, layers=layers, vocab=300, decode_steps=2, seed=960 + B)
    _run_elementwise(oracle, wl, B, N, 2, flags=0x20 if poison else 0, emb_scale=EMB_UNIT, wavefront=True, alibi=alibi, expect_form="groups")


@pytest.mark.parametrize("B,N,layers,d,F,p_min", [(17, 70, 2, 256, 1024, 0), (2, 70, 3, 256, 512, 0), (2, 150, 3, 256, 1024, 64),
                                                  (9, 290, 8, 256, 1024, 0), (9, 100, 8, 256, 1024, 0), (1, 2, 1, 256, 1024, 0), (16, 1, 1, 256, 1024, 0)])
def test_stacks_that_keep_the_launches(oracle, B, N, layers, d, F, p_min):
    """more than sixteen sequences, another hidden width, a wider window, and on either side of where passes over the layers take
    longer than launches that carry all of them: 8 * 290 > 2.75 (290 + 64 * 7), 8 * 100 < 2.75 (100 + 64 * 7); one layer's first positions"""
    wl = gen.Workload("stack_launches", "bf16", B, N, d, d // 64, F, layers=layers, vocab=300, decode_steps=2, seed=970 + B)
    passes, steps = -(-layers // (4 if B <= 4 else 1)) * N, N + 64 * (layers - 1)
    deep = layers > 3 and 100 * passes > 275 * steps
    refused = B > 16 or F != 4 * d or p_min == 64 or layers == 1
    _run_elementwise(oracle, wl, B, N, 2, emb_scale=EMB_UNIT, wavefront=True, p_min=p_min,
                     expect_form="launches" if refused or deep else "groups")


@pytest.mark.parametrize("B,N,d,alibi", [(1, 2, 128, 0.0), (2, 34, 256, 8.0), (3, 65, 384, 0.0), (8, 130, 128, 8.0), (9, 66, 256, 0.0),
                                         (16, 97, 384, 8.0), (4, 290, 256, 0.0), (1, 515, 128, 0.0), (32, 40, 128, 0.0)])
def test_fp32(oracle, B, N, d, alibi):
    """fp32 storage: one sequence per group and several, widths whose share of a contraction ends inside a chunk, blocks of 32 to 512 keys"""
    _run_case(oracle, "f32", B, N, d, d // 64, 4 * d, gains="random", scale=0.5, alpha=0.7, alibi=alibi, kv_cap=N + 1, expect_form="groups")


@pytest.mark.parametrize("B,N,d,F,p_min", [(1, 1, 128, 512, 32), (2, 2, 384, 1536, 32), (33, 40, 128, 512, 32), (17, 40, 384, 1536, 32), (2, 40, 512, 2048, 32), (2, 40, 256, 512, 32), (2, 70, 256, 1024, 16)])
def test_fp32_shapes_that_keep_the_launches(oracle, B, N, d, F, p_min):
    _run_case(oracle, "f32", B, N, d, d // 64, F, p_min=p_min, gains="random", scale=0.5, alpha=0.7, expect_engine="stepwise",
              expect_form="launches")


@pytest.mark.parametrize("d", [256, 512, 768, 1024])
@pytest.mark.parametrize("B,N,alibi", [(1, 33, 8.0), (4, 64, 0.0), (5, 70, 0.0), (8, 34, 8.0)])
def test_reverse_loop(oracle, d, B, N, alibi):
    """the backward pass's loop: one and two sequences per group, full and ragged, blocks of one position and whole ones"""
    _backward_case(oracle, "bf16", B, N, d, d // 64, 4 * d, alpha=0.7, scale=0.125, alibi=alibi, seed=77, expect_form="groups")


def test_reverse_loop_of_nine_sequences(oracle):
    _backward_case(oracle, "bf16", 9, 40, 256, 4, 1024, alpha=0.7, scale=0.125, seed=78, expect_form="launches")


@pytest.mark.parametrize("B,N,d,alibi", [(130, 70, 256, 0.0), (129, 100, 320, 8.0)])
def test_merge_of_eight_lanes_per_row(oracle, B, N, d, alibi):
    """the position-batched merge: windows of 0 to 31 keys, none to two stored levels, heads that do not fill the last workgroup"""
    _run_case(oracle, "bf16", B, N, d, d // 64, 4 * d, gains="random", scale=0.5, alibi=alibi, expect_engine="position-batched")
