"""Contraction gradients at the edges of their staging: reductions of less than, exactly and just past
one and two stages of 64, rows and columns at and past a tile, every shape of the wave grid.
Tolerance as in test_gpu_backward.py (reductions of at most 512 terms)."""
import pytest

from test_gpu_backward import check, make_case, reference, run_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (1, 4, 4, 16, 16),           # one tile, one step of 16
    (63, 4, 4, 16, 64),          # T = 63: no whole stage; K = 64: two waves along the rows
    (64, 4, 4, 64, 80),          # T = 64: one whole stage, nothing left; K = 80: a stage and a step
    (65, 4, 4, 80, 64),          # one tile left over; C = 80: 128-wide columns, ragged
    (128, 4, 4, 128, 128),       # two whole stages, tiles without an edge
    (129, 4, 4, 144, 144),       # a second row block of one tile, a second column block of 16
])
def test_contraction_gradients_at_stage_edges(shape):
    dy, Uq, Vq, scales = make_case(shape, 4, seed=31 + shape[0], per_point=True)
    got = run_backward(dy, Uq, Vq, shape, 4, scales)
    check(reference(dy, Uq, Vq, shape, 4, scales), got, 1e-5)
