"""Flex layers whose work groups hold the channels of one tile (C and K multiples of 256), with the
tiles dealt to XCDs, and layers whose last work group is partly empty: bit-exact against the oracle."""
import pytest

from helpers import small_layer
from oracle import flex, quantised as q
from test_gpu_flex import check, noisy_matrices, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,base,shape,bh,out_type,relu,whole", [
    (4, "legendre", (3, 9, 8, 256, 256), 8, "f32", True, True),      # partial tiles
    (4, "canonical", (9, 8, 8, 256, 256), 8, "i8", False, True),     # 9 images: one past a set of XCDs
    (2, "legendre", (8, 16, 16, 256, 256), 8, "i8", True, True),     # 512 tiles: the aligned eighths
    (6, "legendre", (1, 7, 13, 256, 16), 9, "f32", False, False),    # block-uniform input, per-lane output
    (4, "legendre", (1, 5, 3, 16, 528), 8, "i8", True, False),       # 2 tiles: 4 groups of 256, one of 32
])
def test_flex_layer_of_wide_channels(m, base, shape, bh, out_type, relu, whole):
    xq, wq, s_x, s_w = small_layer(*shape, seed=11 + m)
    fm = noisy_matrices(m, base, seed=m + bh)
    cfg = q.LayerConfig(m=m, base=base, bits_hadamard=bh, out_type=out_type, relu=relu)
    ora, sc = flex.run_layer_flex(xq, wq, s_x, s_w, cfg, fm)
    check(ora, run_gpu(xq, wq, fm, sc, m, base, bh, out_type, relu, whole), out_type)
