"""Batches of more than 32 sequences on the layer-wavefront engine and in multi-launch decoding steps, where the products take
32 sequences per workgroup: one sequence more than a tile, ragged last tiles, contraction shares of one, two, three and four
32-index steps per wavefront, hidden widths that are no multiple of 512, the options of the epilogues."""
import pytest

from paper_2604_21215_amd import inputs as gen
from tests.test_gpu_decode import _decode_case
from tests.test_gpu_parity import _run_case
from tests.test_gpu_stack import EMB_UNIT, _run_elementwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N,d,F,alibi", [(49, 40, 256, 1024, 0.0), (65, 36, 768, 3072, 8.0), (97, 35, 512, 768, 0.0), (128, 34, 1024, 4096, 0.0)])
def test_one_layer_on_the_wavefront_engine(oracle, B, N, d, F, alibi):
    _run_case(oracle, "bf16", B, N, d, d // 64, F, gains="random", scale=0.5, alpha=0.7, kv_cap=N + 1, alibi=alibi, n_decode=2,
              expect_engine="wavefront")


def test_stack_of_33_sequences(oracle):
    wl = gen.Workload("stack_b33", "bf16", 33, 70, 256, 4, 1024, layers=2, vocab=300, decode_steps=2, seed=996)
    _run_elementwise(oracle, wl, 33, 70, 2, emb_scale=EMB_UNIT, wavefront=True)


def test_multi_launch_decode_norm_free_and_single_sequence_tail(oracle):
    _decode_case(oracle, 33, 40, 256, 4, n0=37, steps=[37, 38, 39], seed=61, scale=0.02, flags=1)
