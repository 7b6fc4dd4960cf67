"""Flex backward pass on layers whose images are 1, 2, 4, 8 or 16 tiles: the input bracket's work groups then
take whole images and leave dx themselves.  Against the fp64 oracle; the neighbours of the rule (tiles or
channels that do not fit) take the sum over tiles in a launch of its own."""
import numpy as np
import pytest

from helpers import small_layer
from test_gpu_flex_backward import check, noisy_matrices, oracle_forward, reference, run_gpu

pytestmark = pytest.mark.gpu

CASES = [
    # m, base, (N, H, W, C, K), bits_hadamard
    (4, "legendre", (2, 4, 4, 256, 16), 8),      # 1 tile, 256 channels per work group
    (4, "legendre", (9, 3, 7, 128, 16), 9),      # 2 tiles, ragged
    (4, "canonical", (3, 8, 6, 64, 16), 8),      # 4 tiles
    (2, "legendre", (2, 3, 8, 32, 32), 8),       # 8 tiles
    (4, "legendre", (17, 16, 13, 48, 16), 8),    # 16 tiles, three chunks; two sets of eight images and one more
    (6, "legendre", (2, 19, 24, 16, 16), 8),     # 16 tiles of F(6,3)
    (6, "canonical", (8, 12, 11, 64, 16), 9),    # 4 tiles
    (4, "legendre", (2, 8, 8, 48, 16), 8),       # 4 tiles, channels do not fill 64: per-tile gradients
    (4, "legendre", (2, 12, 12, 32, 16), 8),     # 9 tiles
]


@pytest.mark.parametrize("m,base,shape,bits_hadamard", CASES)
def test_whole_images(m, base, shape, bits_hadamard):
    N, H, W, C, K = shape
    xq, wq, s_x, s_w = small_layer(N, H, W, C, K, seed=1700 + m + C)
    fm = noisy_matrices(m, base, seed=41 + m)
    fwd, sc = oracle_forward(xq, wq, s_x, s_w, fm, m, base, bits_hadamard)
    dy = np.random.default_rng(6 + K).standard_normal((N, H, W, K)).astype(np.float32)
    got = run_gpu(dy, xq, wq, fwd, sc, fm, m, base, bits_hadamard)
    check(reference(dy, xq, wq, fwd, sc, fm, m, base), got)
