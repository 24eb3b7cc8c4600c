"""Batches of more than 32 sequences on the layer-wavefront engine and in multi-launch decoding steps.  From 33 sequences and a width
of 512 on the products take 32 sequences per workgroup: one sequence more than a tile, ragged last tiles, contraction shares of one to
four 32-index steps per wavefront, hidden widths that are no multiple of 512, several layers in a launch, the options of the epilogues.
Narrower layers keep the tiles of 16 sequences."""
import os
import re

import pytest

from paper_2604_21215_amd import inputs as gen
from tests.test_gpu_decode import _decode_case
from tests.test_gpu_parity import _run_case
from tests.test_gpu_stack import EMB_UNIT, _run_elementwise

pytestmark = pytest.mark.gpu


def _takes_wide_products(B, d):
    """the rule of the dispatch, from its source"""
    src = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_21215_amd", "csrc", "rt_wavefront.hip")).read()
    lo_B, lo_d = map(int, re.search(r"constexpr int kWideFrom = (\d+), kWideWidth = (\d+);", src).groups())
    return B >= lo_B and d >= lo_d


@pytest.mark.parametrize("B,N,d,F,alibi", [(49, 40, 256, 1024, 0.0), (65, 36, 768, 3072, 8.0), (97, 35, 512, 768, 0.0), (128, 34, 1024, 4096, 0.0)])
def test_one_layer_on_the_wavefront_engine(oracle, B, N, d, F, alibi):
    _run_case(oracle, "bf16", B, N, d, d // 64, F, gains="random", scale=0.5, alpha=0.7, kv_cap=N + 1, alibi=alibi, n_decode=2,
              expect_engine="wavefront")


def test_stack_of_33_sequences(oracle):
    wl = gen.Workload("stack_b33", "bf16", 33, 70, 256, 4, 1024, layers=2, vocab=300, decode_steps=2, seed=996)
    _run_elementwise(oracle, wl, 33, 70, 2, emb_scale=EMB_UNIT, wavefront=True)


def test_multi_launch_decode_norm_free_and_single_sequence_tail(oracle):
    _decode_case(oracle, 33, 40, 256, 4, n0=37, steps=[37, 38, 39], seed=61, scale=0.02, flags=1)


@pytest.mark.parametrize("B,N,d,F,alibi", [(49, 40, 512, 256, 0.0), (64, 36, 768, 256, 8.0)])
def test_shares_of_one_step(oracle, B, N, d, F, alibi):
    """W2 contracts over 256 indices: one 32-index step per wavefront; 49 sequences leave a tile of one"""
    assert _takes_wide_products(B, d)
    _run_case(oracle, "bf16", B, N, d, d // 64, F, gains="random", scale=0.5, alpha=0.7, kv_cap=N + 1, alibi=alibi, n_decode=2,
              expect_engine="wavefront")


def test_stack_of_33_sequences_wide(oracle):
    """four layers in groups of two: launches over two layers at different positions"""
    assert _takes_wide_products(33, 512)
    wl = gen.Workload("stack_b33_wide", "bf16", 33, 70, 512, 8, 1024, layers=4, vocab=300, decode_steps=2, seed=997)
    _run_elementwise(oracle, wl, 33, 70, 2, emb_scale=EMB_UNIT, wavefront=True)


@pytest.mark.parametrize("flags,gains", [(1, "unit"), (0, "random")])
def test_multi_launch_decode_wide(oracle, flags, gains):
    assert _takes_wide_products(33, 512)
    _decode_case(oracle, 33, 40, 512, 8, n0=37, steps=[37, 38, 39], seed=62, gains=gains, scale=0.02, flags=flags)
