"""Contraction gradients at the edges of their staging: reductions of less than, exactly and just past
one and two stages of 64, rows and columns at and past a tile, every shape of the wave grid.
Tolerance as in test_gpu_backward.py."""
import pytest

from test_gpu_backward import check, make_case, reference, run_backward

pytestmark = pytest.mark.gpu


# shape; whether dV and dU read dM into registers (1) or through LDS (0) (test_launch_rules.py)
CASES = [
    ((1, 4, 4, 16, 16), 0),          # one tile, one step of 16
    ((1, 4, 4, 32, 16), 11),         # the same, from registers
    ((63, 4, 4, 16, 64), 11),        # T = 63: no whole stage; K = 64: two waves along the rows
    ((64, 4, 4, 64, 80), 11),        # T = 64: one whole stage, nothing left; K = 80: a stage and a step
    ((65, 4, 4, 80, 64), 11),        # one tile left over; C = 80: 128-wide columns, ragged
    ((128, 4, 4, 128, 128), 11),     # two whole stages, tiles without an edge
    ((129, 4, 4, 144, 144), 11),     # a second row block of one tile, a second column block of 16
    ((17, 4, 4, 80, 272), 11),       # K = 272: four stages and a step, a third row block of 16
    # more work groups than 384: through LDS, dV where its reduction is short (ranges of 128 tiles)
    ((997, 4, 4, 16, 80), 0),        # 101 tiles in the last range; K = 80: a chunk and half of one
    ((997, 4, 4, 64, 48), 0),
    ((997, 4, 4, 112, 96), 0),
    ((997, 4, 4, 80, 64), 0),
    # ... dU through LDS, dV, whose ranges are long, from registers
    ((2051, 4, 4, 16, 48), 10),      # ranges of 288 tiles, 35 in the last one
    ((2051, 4, 4, 64, 80), 10),
    ((2051, 4, 4, 80, 48), 10),
    ((1025, 4, 4, 208, 144), 10),    # ranges of 288 tiles, 161 in the last one
]


@pytest.mark.parametrize("shape,registers", CASES)
def test_contraction_gradients_at_stage_edges(shape, registers):
    dy, Uq, Vq, scales = make_case(shape, 4, seed=31 + shape[0], per_point=True)
    got = run_backward(dy, Uq, Vq, shape, 4, scales)
    # 3e-5 for the longer reductions, as at 1024 tiles
    check(reference(dy, Uq, Vq, shape, 4, scales), got, 1e-5 if shape[0] <= 512 else 3e-5)
