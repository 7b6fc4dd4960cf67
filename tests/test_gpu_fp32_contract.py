"""The fp32 contraction on the matrix cores (operands cut into three bf16 pieces) against fp64, at the
edges of its tiles: one tile, one row past a tile block, channel counts that fill no chunk or block.

Bound, element by element: the piece products that are left out are together at most 2^-24 of a
product (|m| <= 2^-8 |x|, |l| <= 2^-17 |x|), and its sum of C terms (at most 6 C roundings in fp32, each
2^-24 of a partial sum that never exceeds sum |u v|) adds 6 C 2^-24 sum |u v|."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# m, N, H, W, C, K, blocks per wave along tiles and output channels (test_launch_rules.py)
CASES = [
    (4, 1, 4, 4, 16, 16, 11),        # one tile
    (4, 1, 32, 32, 32, 64, 11),      # 64 tiles
    (4, 1, 20, 52, 48, 80, 11),      # 65 tiles, a partial chunk, K past one 64-wide block
    (4, 1, 32, 64, 144, 128, 11),    # 128 tiles
    (2, 1, 6, 86, 16, 144, 11),      # 129 tiles: one row in the third block
    (6, 3, 23, 37, 80, 48, 11),
    (4, 1, 172, 48, 48, 272, 22),    # 516 tiles: four rows in the last block, a segment of K in the last
    (4, 1, 172, 48, 192, 272, 22),   # the same with U and M past the L2s
    (4, 1, 129, 125, 16, 48, 21),    # 1056 tiles: 32 rows in the last block, K short of one
    (6, 1, 24, 18, 80, 528, 12),     # 12 tiles, a segment of K in the last block
]


@pytest.mark.parametrize("m,N,H,W,C,K,blocks", CASES)
def test_contract_f32_against_fp64(m, N, H, W, C, K, blocks):
    import torch
    import paper_2004_11077_amd as wn
    d = wn.ConvDesc(N, H, W, C, K, m=m, bits_in=32)
    n2, T = d.n ** 2, d.tiles
    rng = np.random.default_rng(7)
    # magnitudes spread over 2^+-12, so that no piece is always the small one
    draw = lambda *s: (rng.standard_normal(s) * 2.0 ** rng.integers(-12, 13, s)).astype(np.float32)
    u, v = draw(n2, T, C), draw(n2, K, C)
    U, V = torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda()
    M = torch.full((n2, T, K), float("nan"), dtype=torch.float32, device="cuda")
    wn.wino_contract(d, U, V, M, wn.Scales.from_dict({}))
    torch.cuda.synchronize()
    u64, v64 = u.astype(np.float64), v.astype(np.float64).transpose(0, 2, 1)
    bound = (6 * C + 1) * 2.0 ** -24 * np.matmul(np.abs(u64), np.abs(v64))
    err = np.abs(M.cpu().numpy().astype(np.float64) - np.matmul(u64, v64))
    assert (err <= bound).all(), float((err / bound).max())


def test_contract_f32_beyond_the_range_of_its_pieces():
    """Infinities, NaNs and values past the largest bf16 give what plain fp32 sums give."""
    import torch
    import paper_2004_11077_amd as wn
    d = wn.ConvDesc(1, 4, 20, 48, 80, m=4, bits_in=32)
    n2, T, C, K = d.n ** 2, d.tiles, 48, 80
    rng = np.random.default_rng(11)
    u = rng.standard_normal((n2, T, C)).astype(np.float32)
    v = rng.uniform(0.5, 1.0, (n2, K, C)).astype(np.float32)
    u[0, 0, 3], u[1, 1, 40], u[2, 2, 7] = np.inf, -np.inf, np.nan
    u[3, 3, 0], u[3, 3, 1] = np.inf, -np.inf
    u[4, 4, 5] = 3.4e38                       # finite, rounds to an infinite bf16
    v[5, 6, 7] = np.inf
    M = torch.full((n2, T, K), 7.0, dtype=torch.float32, device="cuda")
    wn.wino_contract(d, torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda(), M,
                     wn.Scales.from_dict({}))
    torch.cuda.synchronize()
    got = M.cpu().numpy()
    with np.errstate(all="ignore"):
        # channel by channel: a library product of non-finite matrices may take any order
        want = sum(u[..., None, c].astype(np.float64) * v[:, None, :, c] for c in range(C))
    assert np.isinf(want[0, 0]).all() and np.isnan(want[2, 2]).all() and np.isnan(want[3, 3]).all()
    for cls in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(cls(got), cls(want)), cls
    ok = np.isfinite(want)
    size = sum(np.abs(u[..., None, c].astype(np.float64) * v[:, None, :, c]) for c in range(C))
    bound = (6 * C + 1) * 2.0 ** -24 * size
    assert (np.abs(got[ok] - want[ok]) <= bound[ok]).all()


@pytest.mark.parametrize("eu,ev", [
    (-124, 0),       # low pieces of u far below the smallest bf16
    (-126, 20),      # the smallest normal numbers
    (-140, 30),      # subnormal u
    (0, -135),       # subnormal v
    (-124, 110),     # tiny times large: an ordinary result
    (-70, -70),      # subnormal result
])
def test_contract_f32_of_tiny_operands(eu, ev):
    """Operands far below one keep all their 24 bits (what a subnormal has of them).  Bound as above,
    plus half the smallest subnormal where the result is stored, and where a plain sum adds one (C of
    them)."""
    import torch
    import paper_2004_11077_amd as wn
    d = wn.ConvDesc(1, 12, 44, 48, 80, m=4, bits_in=32)
    n2, T, C, K = d.n ** 2, d.tiles, 48, 80
    rng = np.random.default_rng(5)
    u = np.ldexp(rng.uniform(-1, 1, (n2, T, C)), eu).astype(np.float32)
    v = np.ldexp(rng.uniform(-1, 1, (n2, K, C)), ev).astype(np.float32)
    M = torch.full((n2, T, K), float("nan"), dtype=torch.float32, device="cuda")
    wn.wino_contract(d, torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda(), M,
                     wn.Scales.from_dict({}))
    torch.cuda.synchronize()
    u64, v64 = u.astype(np.float64), v.astype(np.float64).transpose(0, 2, 1)
    bound = (6 * C + 1) * 2.0 ** -24 * np.matmul(np.abs(u64), np.abs(v64)) + (C + 1) * 2.0 ** -150
    err = np.abs(M.cpu().numpy().astype(np.float64) - np.matmul(u64, v64))
    assert (err <= bound).all(), float((err / bound).max())


@pytest.mark.parametrize("N,H,W,C,K", [
    (1, 4, 4, 16, 16),           # one tile
    (1, 20, 52, 48, 80),         # 65 tiles, a partial chunk, K past one 64-wide block
    (1, 86, 24, 144, 144),       # 132 tiles: four rows and one 16-wide segment past a work group
    (1, 172, 48, 48, 272),       # the same past work groups of twice the rows and columns
])
def test_work_groups_with_sums_that_are_not_finite(N, H, W, C, K):
    """Plain fp32 sums at the edges of a work group's tile: an infinity in the last channel of the last
    tile, a NaN in the last filter, a point whose operands and sums are beyond the scaled range."""
    import torch
    import paper_2004_11077_amd as wn
    d = wn.ConvDesc(N, H, W, C, K, m=4, bits_in=32)
    n2, T = d.n ** 2, d.tiles
    rng = np.random.default_rng(C)
    u = rng.standard_normal((n2, T, C)).astype(np.float32)
    v = rng.uniform(0.5, 1.0, (n2, K, C)).astype(np.float32)
    u[0, -1, -1], v[1, -1, 0] = np.inf, np.nan
    u[2] *= np.float32(2.0 ** 115)
    M = torch.full((n2, T, K), 7.0, dtype=torch.float32, device="cuda")
    wn.wino_contract(d, torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda(), M,
                     wn.Scales.from_dict({}))
    torch.cuda.synchronize()
    got = M.cpu().numpy().astype(np.float64)
    u64, v64 = u.astype(np.float64), v.astype(np.float64).transpose(0, 2, 1)
    assert np.isposinf(got[0, -1]).all() and np.isnan(got[1, :, -1]).all()
    ok = np.ones(got.shape, bool)
    ok[0, -1], ok[1, :, -1] = False, False
    u64[0, -1, -1], v64[1, 0, -1] = 0.0, 0.0
    bound = (6 * C + 1) * 2.0 ** -24 * np.matmul(np.abs(u64), np.abs(v64))
    err = np.abs(got - np.matmul(u64, v64), where=ok, out=np.zeros_like(got))
    assert (err <= bound).all()
