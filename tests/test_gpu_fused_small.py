"""The single-kernel layer at every number of tiles per work group (16, 8, 4, by the size of the grid),
with filters transformed inside it (few filters) or before it, and with several blocks of output
channels: bit-exact against the oracle, the filters it leaves in the workspace included."""
import pytest

from helpers import assert_layer_parity, gpu_layer, oracle_layer, small_layer

pytestmark = pytest.mark.gpu


# m, base, bits of M, output, relu, per point, shape, tiles per work group (test_launch_rules.py)
CASES = [
    (4, "legendre", 8, "f32", False, False, (1, 3, 5, 16, 16), 4),      # 2 tiles, own filters
    (2, "canonical", 9, "i8", True, False, (1, 9, 9, 16, 64), 4),       # 25 tiles: one in the last group of 4
    (4, "legendre", 9, "i8", False, True, (3, 9, 5, 32, 32), 4),        # 1024 filters: the most it takes
    (4, "legendre", 8, "i8", True, False, (2, 9, 9, 16, 80), 4),        # 1280 filters: transformed before it
    (2, "legendre", 8, "f32", True, True, (1, 61, 66, 48, 16), 4),      # 1023 tiles
    (4, "canonical", 8, "i8", False, False, (1, 132, 132, 16, 16), 8),  # 1089 tiles: one in the last group
    (2, "legendre", 9, "i8", True, False, (1, 131, 129, 16, 16), 8),    # 4290 tiles: two in the last group
    (4, "legendre", 8, "i8", True, False, (1, 12, 20, 64, 208), 4),     # four blocks of output channels
    (4, "canonical", 9, "f32", False, False, (1, 7, 9, 64, 144), 4),    # five blocks of 32
    # 8177 tiles: one in the last group of 16
    (4, "legendre", 8, "i8", True, False, (13, 66, 146, 16, 16), 16),
    (2, "canonical", 8, "f32", False, True, (13, 33, 73, 48, 16), 16),  # three of four segments of channels
    (4, "canonical", 9, "f32", True, False, (13, 65, 147, 16, 16), 16),
    (2, "legendre", 9, "i8", False, True, (7, 22, 106, 32, 64), 16),    # 4081 tiles, two blocks of 32
    (4, "legendre", 9, "i8", False, True, (13, 66, 146, 16, 16), 16),
]


@pytest.mark.parametrize("m,base,bh,out_type,relu,pp,shape,tiles", CASES)
def test_single_kernel_layer(m, base, bh, out_type, relu, pp, shape, tiles):
    xq, wq, s_x, s_w = small_layer(*shape, seed=17 + m + bh, outliers=0.01 if pp else 0.0)
    kw = dict(m=m, base=base, bits_hadamard=bh, out_type=out_type, relu=relu)
    ora, sc = oracle_layer(xq, wq, s_x, s_w, per_point=pp, **kw)
    assert_layer_parity(ora, gpu_layer(xq, wq, sc, fused=True, **kw), out_type)


def test_small_layers_take_one_launch():
    import paper_2004_11077_amd as wn
    auto = dict(m=4, fused=wn.FUSED_AUTO)
    assert wn.wino_conv2d_launches(wn.ConvDesc(1, 8, 8, 16, 16, **auto)) == ["fused_layer"]
    assert wn.wino_conv2d_launches(wn.ConvDesc(8, 8, 8, 64, 128, weights_pretransformed=1, **auto)) == ["fused_layer"]
    assert wn.wino_conv2d_launches(wn.ConvDesc(1, 8, 8, 16, 80, **auto)) == ["weight_transform", "fused_layer"]
