"""The integer brackets on the matrix pipe (F(4,3), Legendre base, one scale per tensor): the input
transform, the contraction + output kernel and the single kernel, bit-exact against the oracle at
the edges of their blocks, and where their rules send a layer to the general form."""
import numpy as np
import pytest

from helpers import assert_layer_parity, gpu_layer, oracle_layer, small_layer

pytestmark = pytest.mark.gpu

# bits of M, output, relu, shape, tiles per work group of the single kernel (test_matrix_rules.py)
FUSED_CASES = [
    (8, "f32", True, (1, 17, 6, 16, 96), 4),          # 10 tiles, a partial second block of channels
    (9, "i8", False, (2, 13, 9, 48, 48), 4),          # 24 tiles, half a block of 32
    (8, "i8", True, (1, 148, 148, 16, 16), 8),        # 1369 tiles: one in the last group
    (9, "f32", True, (1, 132, 132, 16, 32), 8),       # 1089 tiles: one in the last group
    (8, "f32", False, (13, 66, 146, 32, 48), 16),     # 8177 tiles: one in the last group
    (9, "i8", True, (13, 65, 147, 16, 32), 16),
]


@pytest.mark.parametrize("bh,out_type,relu,shape,tiles", FUSED_CASES)
def test_single_kernel(bh, out_type, relu, shape, tiles):
    xq, wq, s_x, s_w = small_layer(*shape, seed=5 + bh + tiles, outliers=0.01)
    kw = dict(m=4, base="legendre", bits_hadamard=bh, out_type=out_type, relu=relu)
    ora, sc = oracle_layer(xq, wq, s_x, s_w, **kw)
    assert_layer_parity(ora, gpu_layer(xq, wq, sc, fused=True, **kw), out_type)


def operands(x, w, sc, frag):
    import torch
    import paper_2004_11077_amd as wn
    N, H, W, C = x.shape
    d = wn.ConvDesc(N, H, W, C, w.shape[0], m=4, base=wn.BASE_LEGENDRE,
                    operand_layout=wn.LAYOUT_FRAGMENTS if frag else wn.LAYOUT_ROWS)
    vb, ub = wn.wino_operand_bytes(d)
    U = torch.full((ub,), 77, dtype=torch.int8, device="cuda:0")
    V = torch.full((vb,), 77, dtype=torch.int8, device="cuda:0")
    wn.wino_transform_operands(d, x, U, w, V, sc)
    U2 = torch.full((ub,), 77, dtype=torch.int8, device="cuda:0")
    wn.wino_input_transform(d, x, U2, sc)
    assert torch.equal(U, U2)
    u = U.cpu().numpy()
    return wn.defragment(u, d.n ** 2, d.tiles, C) if frag else u.reshape(d.n ** 2, d.tiles, C)


# the last one: rows of 65536 bytes; all of them few enough items for the general form
@pytest.mark.parametrize("frag", [False, True])
@pytest.mark.parametrize("shape", [(1, 4, 4, 16), (3, 5, 6, 48), (1, 9, 13, 80), (5, 4, 4, 256), (2, 7, 9, 272),
                                   (1, 4, 4096, 16)])
def test_input_transform(shape, frag):
    import torch
    import paper_2004_11077_amd as wn
    xq, wq, s_x, s_w = small_layer(*shape, 16, seed=3)
    xq.reshape(-1)[:shape[3]] = -127                      # the most negative code of a cast
    ora, sc = oracle_layer(xq, wq, s_x, s_w, m=4, base="legendre")
    dev = torch.device("cuda:0")
    x, w = (torch.from_numpy(np.ascontiguousarray(v, dtype=np.int8)).to(dev) for v in (xq, wq))
    assert np.array_equal(operands(x, w, wn.Scales.from_dict(sc), frag), ora["U"])


# enough items for the matrix pipe (test_matrix_rules.py): images of one tile, ragged edges, channels that do not fill 64,
# whole tiles with an odd number of blocks, a partial last block, rows of nearly 65536 bytes
MATRIX_INPUTS = [(6145, 4, 4, 16), (513, 9, 13, 16), (260, 5, 15, 48), (193, 7, 9, 128), (385, 4, 4, 256), (65, 7, 9, 272),
                 (129, 6, 8, 512), (1, 27, 4095, 16)]


@pytest.mark.parametrize("frag", [False, True])
@pytest.mark.parametrize("shape", MATRIX_INPUTS)
def test_input_transform_on_the_matrix_pipe(shape, frag):
    test_input_transform(shape, frag)


# the tallest image of the matrix pipe, and two whose last tiles reach row 65536: beyond sixteen bits it would count
# as row 0, and the next image's rows would be read for padding; rows of 65536 bytes, which the general form takes too
@pytest.mark.parametrize("H,W", [(65532, 4), (65533, 4), (65534, 4), (27, 4096)])
def test_input_transform_large_images(H, W):
    import torch
    import paper_2004_11077_amd as wn
    from oracle import quantised as q
    rng = np.random.default_rng(H)
    xq = rng.integers(-127, 128, (2, H, W, 16)).astype(np.int8)
    wq = rng.integers(-127, 128, (16, 16, 3, 3)).astype(np.int8)
    cfg, sc = q.LayerConfig(m=4, base="legendre"), dict(s_w=0.01, s_w1=0.02, s_v=0.05, s_m=1.0, s_m1=1.0, s_y=1.0)
    want = q.input_transform(xq, np.float32(0.02), cfg, q.StageMatrices(cfg), sc, {})
    x, w = (torch.from_numpy(v).to("cuda:0") for v in (xq, wq))
    assert np.array_equal(operands(x, w, wn.Scales.from_dict(dict(sc, s_x=0.02)), False), want)


@pytest.mark.parametrize("frag,shape", [(False, (1025, 8, 8, 256)), (True, (1100, 8, 8, 192)), (False, (2101, 8, 8, 144))])
def test_input_transform_work_groups_take_several_blocks(frag, shape):
    """More blocks than work groups; every image's tiles come out as in a batch of eight images."""
    import torch
    import paper_2004_11077_amd as wn
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    x = torch.randint(-128, 128, shape, generator=gen, dtype=torch.int8, device="cuda:0")
    w = torch.randint(-127, 128, (16, shape[3], 3, 3), generator=gen, dtype=torch.int8, device="cuda:0")
    sc = wn.Scales.from_dict(dict(s_x=0.02, s_w=0.01, s_x1=0.03, s_w1=0.02, s_u=0.1, s_v=0.05, s_m=1.0, s_m1=1.0))
    u = operands(x, w, sc, frag)
    step = 8
    for n in list(range(0, shape[0], 97 * step // 8)) + [shape[0] - step]:
        part = operands(x[n:n + step].contiguous(), w, sc, frag)
        assert np.array_equal(part, u[:, 4 * n:4 * n + part.shape[1]]), n


@pytest.mark.parametrize("bh", [8, 9])
@pytest.mark.parametrize("C", [32, 144])
def test_output_scale_beyond_the_scaled_multipliers(bh, C):
    """A dequantisation factor that 2^24 would take out of fp32: the general form, same values as the stages."""
    xq, wq, s_x, s_w = small_layer(2, 9, 10, C, 48, seed=9)
    kw = dict(m=4, base="legendre", bits_hadamard=bh)
    _, sc = oracle_layer(xq, wq, s_x, s_w, **kw)
    for factor in (2.0 ** 90, 2.0 ** 118):
        big = dict(sc, **{k: sc[k] * factor for k in ("s_x", "s_x1", "s_u", "s_m", "s_m1")})
        with np.errstate(over="ignore"):
            a = gpu_layer(xq, wq, big, **kw)["y"]
            b = gpu_layer(xq, wq, big, fused=True, **kw)["y"]
        assert np.abs(a).max() > 1e20 and np.array_equal(a, b, equal_nan=True)


# (images of one tile, ragged edges, partial last blocks of 128 and 256 items; more pairs of blocks than work groups)
@pytest.mark.parametrize("shape", [(1, 4, 4, 16, 16), (3, 5, 7, 16, 48), (9, 3, 2, 16, 80), (5, 4, 4, 16, 256), (2, 18, 5, 16, 272)])
@pytest.mark.parametrize("out_type,relu", [("f32", False), ("i8", True)])
def test_output_transform(shape, out_type, relu):
    xq, wq, s_x, s_w = small_layer(*shape, seed=13)
    kw = dict(m=4, base="legendre", out_type=out_type, relu=relu)
    ora, sc = oracle_layer(xq, wq, s_x, s_w, **kw)
    assert_layer_parity(ora, gpu_layer(xq, wq, sc, **kw), out_type)


# The whole batch and eight of its images at a time: several blocks per work group (513 and 1030 images), and batches on
# either side of the lines between the two forms (OUTPUT_LINES in test_matrix_rules.py).
@pytest.mark.parametrize("N,H,W,K,out_type", [
    (513, 16, 16, 208, "f32"), (1030, 8, 8, 256, "f32"), (1030, 8, 8, 256, "i8"),
    (1536, 8, 8, 64, "f32"), (1537, 8, 8, 64, "f32"), (4095, 8, 8, 64, "f32"), (4096, 8, 8, 64, "f32"),
    (8192, 8, 8, 64, "f32"), (8192, 8, 8, 64, "i8"), (2048, 8, 8, 256, "i8"), (2049, 8, 8, 256, "i8")])
def test_output_transform_work_groups_take_several_blocks(N, H, W, K, out_type):
    import torch
    import paper_2004_11077_amd as wn
    sc = wn.Scales.from_dict(dict(s_x=0.02, s_w=0.01, s_x1=0.03, s_w1=0.02, s_u=0.1, s_v=0.05, s_m=1.0, s_m1=1.5, s_y=20.0))
    gen = torch.Generator(device="cuda:0").manual_seed(2)
    per = (H // 4) * (W // 4)
    M = torch.randint(-127, 128, (36, N * per, K), generator=gen, dtype=torch.int8, device="cuda:0")

    def outputs(m, n):
        d = wn.ConvDesc(n, H, W, 16, K, m=4, base=wn.BASE_LEGENDRE,
                        out_type=wn.OUT_I8 if out_type == "i8" else wn.OUT_F32)
        y = torch.full((n, H, W, K), 7, dtype=torch.int8 if out_type == "i8" else torch.float32, device="cuda:0")
        return wn.wino_output_transform(d, m, y, sc)

    y = outputs(M, N)
    for n in list(range(0, N - 8, 61)) + [N - 8]:
        part = outputs(M[:, n * per:(n + 8) * per].contiguous(), 8)
        assert torch.equal(part, y[n:n + 8]), n
