"""Quantised contraction against exact integers at the edges of its tiles and chunks: one tile, a row
past a block, channel counts of less than a chunk of 128, one chunk, and a chunk and a rest, filters
that fill no block.  Codes must be equal."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# shape, tile rows of a work group (64 unless 128-row blocks are many; test_launch_rules.py)
CASES = [
    ((1, 4, 4, 16, 16), 64),
    ((33, 4, 4, 112, 144), 64),  # 33 tiles, 7 of 8 segments of a chunk, a block and one segment of filters
    ((1, 32, 32, 128, 80), 64),  # 64 tiles, exactly a chunk
    ((65, 4, 4, 144, 128), 64),  # 65 tiles, a chunk and a segment
    ((1, 172, 48, 272, 48), 64),    # 516 tiles: eight blocks and four rows, two chunks and a segment
    ((1, 172, 48, 144, 272), 128),  # 516 tiles: four blocks and four rows, two blocks of filters and a segment
    ((15, 44, 44, 48, 16), 128),    # 1815 tiles: 14 blocks and 23 rows, less than a chunk, one segment of filters
]


@pytest.mark.parametrize("hadamard", [8, 9])
@pytest.mark.parametrize("shape,rows", CASES)
def test_contract_codes(shape, rows, hadamard):
    N, H, W, C, K = shape
    import torch
    import paper_2004_11077_amd as wn
    d = wn.ConvDesc(N, H, W, C, K, m=4, bits_hadamard=hadamard)
    n2, T, q = d.n ** 2, d.tiles, 127 if hadamard == 8 else 255
    rng = np.random.default_rng(C + K)
    u = rng.integers(-127, 128, (n2, T, C)).astype(np.int8)
    v = rng.integers(-127, 128, (n2, K, C)).astype(np.int8)
    real = np.matmul(u.astype(np.float64), v.astype(np.float64).transpose(0, 2, 1))   # exact
    s_m = float(np.float32(np.abs(real).max() / q))
    sc = wn.Scales.from_dict({"s_u": 1.0, "s_v": 1.0, "s_m": s_m})
    M = torch.full((n2, T, K), 99, dtype=torch.int8 if hadamard == 8 else torch.int16, device="cuda")
    wn.wino_contract(d, torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda(), M, sc)
    torch.cuda.synchronize()
    # the cast rounds the exact product of two fp32 numbers once
    mult = np.float64(np.float32(1.0 / np.float64(np.float32(s_m))))
    want = np.clip(np.rint(real * mult), -q, q).astype(np.int32)
    assert np.array_equal(M.cpu().numpy().astype(np.int32), want)
