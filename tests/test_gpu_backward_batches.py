"""rt_layer_backward with more sequences than the single-launch reverse loop takes: the loop's products on the matrix cores from
three bf16 parts of their fp32 inputs, at the edges of their tiles (16 sequences, 16 or 32 outputs) and contraction pieces (64
indices over eight wavefronts: fewer pieces than wavefronts, whole groups, a ragged last group)."""
import pytest

from tests.test_gpu_backward import _run

pytestmark = pytest.mark.gpu

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
