"""Tensors that start between 16-byte boundaries, in the calls that take them there: the stages of a layer
with run-time matrices (any byte, fp32 y any float) and the fp32 path (any float).  Results must equal
those of aligned tensors bit for bit."""
import numpy as np
import pytest

from helpers import small_layer
from oracle import flex, quantised as q
from test_gpu_flex import noisy_matrices

pytestmark = pytest.mark.gpu


def at(t, shift):
    """A copy of t that starts `shift` elements past a 256-byte boundary, between guard elements."""
    import torch
    buf = torch.full((t.numel() + shift + 64,), 85, dtype=t.dtype, device="cuda")
    v = buf[shift:shift + t.numel()].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 256 == shift * t.element_size()
    return v, buf


def intact(v, buf, shift):
    return bool((buf[:shift] == 85).all()) and bool((buf[shift + v.numel():] == 85).all())


@pytest.mark.parametrize("shift", [1, 8, 15])
@pytest.mark.parametrize("m,base,bh,out_type,shape", [
    (4, "legendre", 8, "i8", (3, 9, 10, 48, 80)),        # partly empty last work group
    (2, "canonical", 8, "f32", (2, 8, 6, 256, 256)),     # one tile per work group
    (6, "legendre", 9, "f32", (1, 7, 13, 32, 16)),
])
def test_flex_stages_at_any_byte(m, base, bh, out_type, shape, shift):
    import torch
    import paper_2004_11077_amd as wn
    N, H, W, C, K = shape
    xq, wq, s_x, s_w = small_layer(*shape, seed=60 + m)
    fm = noisy_matrices(m, base, seed=m)
    cfg = q.LayerConfig(m=m, base=base, bits_hadamard=bh, out_type=out_type)
    ora, scales = flex.run_layer_flex(xq, wq, s_x, s_w, cfg, fm)
    desc = wn.ConvDesc(N, H, W, C, K, m=m, bits_hadamard=bh,
                       base=wn.BASE_LEGENDRE if base == "legendre" else wn.BASE_CANONICAL,
                       out_type=wn.OUT_I8 if out_type == "i8" else wn.OUT_F32)
    gfm, sc = wn.FlexMatrices(fm.GP, fm.BPT, fm.APT), wn.Scales.from_dict(scales)
    n2, T = desc.n ** 2, desc.tiles
    new = lambda *s, dt=torch.int8: torch.zeros(s, dtype=dt)
    x, xb = at(torch.from_numpy(xq), shift)
    w, wb = at(torch.from_numpy(wq), shift)
    V, Vb = at(new(n2, K, C), shift)
    U, Ub = at(new(n2, T, C), shift)
    Mb = torch.zeros((n2, T, K), dtype=torch.int8 if bh == 8 else torch.int16, device="cuda")
    y, yb = at(new(N, H, W, K, dt=torch.int8 if out_type == "i8" else torch.float32), shift)
    wn.wino_flex_weight_transform(desc, gfm, w, V, sc)
    wn.wino_flex_input_transform(desc, gfm, x, U, sc)
    wn.wino_contract(desc, U.clone(), V.clone(), Mb, sc)     # takes multiples of 16 only
    M, Mbuf = at(Mb, shift)
    wn.wino_flex_output_transform(desc, gfm, M, y, sc)
    torch.cuda.synchronize()
    for name, t in (("V", V), ("U", U), ("M", M), ("y", y)):
        want = ora[name].astype(np.float32) if name == "y" and out_type == "f32" else ora[name]
        assert np.array_equal(t.cpu().numpy().astype(want.dtype), want), name
    for v, buf in ((V, Vb), (U, Ub), (y, yb)):
        assert intact(v, buf, shift)
    # the whole layer and the choice of its scales, from the same x and w
    ws = torch.empty(wn.wino_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    y.zero_()
    wn.wino_flex_conv2d(desc, gfm, x, w, y, sc, ws)
    cal = torch.empty(wn.wino_calibrate_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    got = wn.wino_flex_calibrate(desc, gfm, x, w, None, float(s_x), float(s_w), cal)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy().astype(want.dtype), want)
    for name, val in scales.items():
        if name != "s_y":
            assert np.float32(getattr(got, name)) == np.float32(val), name


@pytest.mark.parametrize("shift", [1, 3])
def test_fp32_path_at_any_float(shift):
    import torch
    import paper_2004_11077_amd as wn
    N, H, W, C, K = 2, 10, 23, 48, 80
    desc = wn.ConvDesc(N, H, W, C, K, m=4, bits_in=32)
    n2, T = desc.n ** 2, desc.tiles
    gen = torch.Generator().manual_seed(2)
    x, w = torch.randn((N, H, W, C), generator=gen), torch.randn((K, C, 3, 3), generator=gen)
    none = wn.Scales.from_dict({})

    def run(shift):
        parts = [at(t, shift) for t in (x, w, torch.zeros(n2, T, C), torch.zeros(n2, K, C),
                                        torch.zeros(n2, T, K), torch.zeros(N, H, W, K))]
        xv, wv, U, V, M, y = (v for v, _ in parts)
        wn.wino_input_transform(desc, xv, U, none)
        wn.wino_weight_transform(desc, wv, V, none)
        wn.wino_contract(desc, U, V, M, none)
        wn.wino_output_transform(desc, M, y, none)
        torch.cuda.synchronize()
        assert all(intact(v, buf, shift) for v, buf in parts)
        return [t.cpu().numpy() for t in (U, V, M, y)]

    for a, b in zip(run(0), run(shift)):
        assert np.array_equal(a, b)
