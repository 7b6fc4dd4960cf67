"""Scales of a flex layer chosen on the device, at the ends of the range: one tile and 16 channels (the
smallest scratch region), several work groups with a partly empty last one, contractions in blocks of 64 and
of 128 rows, all widths of M in both bases.  Every scale and the output must equal the oracle's bit for bit."""
import numpy as np
import pytest

from helpers import small_layer
from oracle import flex, quantised as q
from test_gpu_flex import noisy_matrices

pytestmark = pytest.mark.gpu


CASES = [
    (2, "legendre", 8, "f32", False, (1, 2, 2, 16, 16)),
    (4, "legendre", 9, "i8", True, (1, 3, 4, 16, 16)),
    (6, "canonical", 9, "i8", False, (1, 6, 6, 16, 16)),
    (4, "legendre", 8, "f32", True, (3, 13, 10, 48, 80)),
    (6, "legendre", 32, "f32", False, (2, 7, 13, 32, 48)),
    (4, "canonical", 32, "i8", True, (2, 9, 9, 80, 144)),
    (2, "canonical", 8, "i8", True, (9, 8, 8, 16, 256)),
]
# at least 512 blocks of 128 rows: the contraction's other block height (test_launch_rules.py), with
# ragged tiles and filters
WIDE_CASES = [
    (4, "legendre", 8, "i8", True, (1, 172, 48, 16, 272)),      # 516 tiles: four rows in the last block
    (4, "canonical", 9, "f32", False, (1, 172, 48, 16, 272)),
    (6, "legendre", 9, "i8", False, (1, 78, 120, 16, 272)),     # 260 tiles
    (2, "canonical", 8, "f32", True, (3, 39, 70, 32, 528)),     # 2100 tiles: 52 rows in the last block
]


@pytest.mark.parametrize("m,base,bh,out_type,relu,shape", CASES + WIDE_CASES)
def test_device_chosen_scales_equal_the_oracles(m, base, bh, out_type, relu, shape):
    import torch
    import paper_2004_11077_amd as wn
    N, H, W, C, K = shape
    xq, wq, s_x, s_w = small_layer(N, H, W, C, K, seed=400 + m)
    fm = noisy_matrices(m, base, seed=m + 50)
    cfg = q.LayerConfig(m=m, base=base, bits_hadamard=bh, out_type=out_type, relu=relu)
    ora, sc = flex.run_layer_flex(xq, wq, s_x, s_w, cfg, fm)
    desc = wn.ConvDesc(N, H, W, C, K, m=m, bits_hadamard=bh, relu=int(relu),
                       base=wn.BASE_LEGENDRE if base == "legendre" else wn.BASE_CANONICAL,
                       out_type=wn.OUT_I8 if out_type == "i8" else wn.OUT_F32)
    x, w = torch.from_numpy(xq).cuda(), torch.from_numpy(wq).cuda()
    y = torch.zeros((N, H, W, K), dtype=torch.int8 if out_type == "i8" else torch.float32, device="cuda")
    ws = torch.randint(0, 255, (wn.wino_calibrate_workspace_bytes(desc),), dtype=torch.uint8, device="cuda")
    got = wn.wino_flex_calibrate(desc, wn.FlexMatrices(fm.GP, fm.BPT, fm.APT), x, w, y, float(s_x),
                                 float(s_w), ws)
    torch.cuda.synchronize()
    for name, val in sc.items():
        assert np.float32(getattr(got, name)) == np.float32(val), name
    assert np.array_equal(y.cpu().numpy(), ora["y"].astype(np.int8 if out_type == "i8" else np.float32))


@pytest.mark.parametrize("m,base,bh,s_x,s_w,size,bad", [
    (4, "legendre", 8, 0.1, 1e-45, 0.01, "s_w1"),      # the filters' scales underflow
    (4, "canonical", 8, 0.1, 3e38, 1000.0, "s_v"),     # and overflow
    (2, "legendre", 9, 3e38, 0.1, 1000.0, "s_x1"),     # those of the activations
    (4, "canonical", 8, 1e-45, 0.1, 0.01, "s_u"),
    (2, "canonical", 9, 1e-25, 1e-25, 1.0, "s_m"),     # the product of two good ones underflows
])
@pytest.mark.parametrize("with_y", [False, True])
def test_scales_that_no_stage_call_takes_are_refused(m, base, bh, s_x, s_w, size, bad, with_y):
    """A chosen scale that underflows to zero or overflows is an error of the calibration, whether or
    not an output is asked for."""
    import torch
    import paper_2004_11077_amd as wn
    N, H, W, C, K = 1, 9, 9, 16, 16
    xq, wq, _, _ = small_layer(N, H, W, C, K, seed=3)
    fm = noisy_matrices(m, base, seed=1)
    desc = wn.ConvDesc(N, H, W, C, K, m=m, bits_hadamard=bh,
                       base=wn.BASE_LEGENDRE if base == "legendre" else wn.BASE_CANONICAL)
    x, w = torch.from_numpy(xq).cuda(), torch.from_numpy(wq).cuda()
    y = torch.zeros((N, H, W, K), dtype=torch.float32, device="cuda") if with_y else None
    ws = torch.empty(wn.wino_calibrate_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    gfm = wn.FlexMatrices(*(np.float32(size) * a for a in (fm.GP, fm.BPT, fm.APT)))
    with pytest.raises(wn.WinoError, match="bad .*" + bad):
        wn.wino_flex_calibrate(desc, gfm, x, w, y, s_x, s_w, ws)
    torch.cuda.synchronize()
    # the same call with ordinary scales goes through
    sc = wn.wino_flex_calibrate(desc, wn.FlexMatrices(fm.GP, fm.BPT, fm.APT), x, w, y, 0.1, 0.1, ws)
    assert 0 < sc.s_u < np.inf and 0 < sc.s_v < np.inf and 0 < sc.s_m < np.inf


def test_calibrations_on_several_threads_and_streams():
    """More threads than read-back buffers, each with a layer and a stream of its own: every one gets its scales."""
    import threading
    import torch
    import paper_2004_11077_amd as wn
    fm = noisy_matrices(4, "legendre", seed=9)
    gfm = wn.FlexMatrices(fm.GP, fm.BPT, fm.APT)
    desc = wn.ConvDesc(2, 9, 9, 16, 16, m=4, base=wn.BASE_LEGENDRE)
    calls = []
    for i in range(10):
        xq, wq, s_x, s_w = small_layer(2, 9, 9, 16, 16, seed=60 + i)
        x, w = torch.from_numpy(xq).cuda(), torch.from_numpy(wq).cuda()
        ws = torch.empty(wn.wino_calibrate_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
        calls.append((desc, gfm, x, w, None, float(s_x) * (i + 1), float(s_w), ws, torch.cuda.Stream()))
    torch.cuda.synchronize()

    def scales(call):
        sc = wn.wino_flex_calibrate(*call)
        return [getattr(sc, k) for k in wn.Scales.SCALARS]

    want = [scales(c) for c in calls]
    got = [[] for _ in calls]
    threads = [threading.Thread(target=lambda i=i: got[i].extend(scales(calls[i]) for _ in range(25)))
               for i in range(len(calls))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len({tuple(v) for v in want}) == len(calls)
    assert all(len(g) == 25 and all(v == w for v in g) for g, w in zip(got, want))
