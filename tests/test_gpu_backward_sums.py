"""Gain gradients of rt_layer_backward at the edges of their row slices (32 rows and up, 64 slices at most): fewer rows than
a slice, one row more than whole slices, more rows than 64 slices of 32."""
import pytest

from tests.test_gpu_backward import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N", [(1, 5), (1, 33), (3, 43), (3, 683), (2, 1025)])
def test_gain_gradients_row_slices(oracle, B, N):
    _run(oracle, "f32", B, N, 64, 1, 128, scale=0.25, alpha=0.7)
