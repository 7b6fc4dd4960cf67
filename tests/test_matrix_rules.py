"""The work groups that the GPU tests of the matrix-pipe brackets name, against the library's rule; the
dealing of two-block work groups to XCDs is one-to-one."""
import test_gpu_matrix_brackets as brackets
from test_host_indexing import needs_hipcc, run_host_program

pytestmark = needs_hipcc


def test_single_kernel_cases_run_the_group_they_name(tmp_path):
    args = [str(v) for bh, _, _, (N, H, W, C, K), _ in brackets.FUSED_CASES for v in (N, H, W, K, bh)]
    got = [int(v) for v in run_host_program(tmp_path, "matrix_rules", args)]
    want = [c[4] for c in brackets.FUSED_CASES]
    assert got == want and set(want) == {4, 8, 16}


def test_dealing_of_block_pairs(tmp_path):
    assert run_host_program(tmp_path, "pair_dealing")[0] == "ok"


def test_sixteen_bit_pixel_coordinates(tmp_path):
    """Tiles reach past the image: 65532 rows are the most whose padding rows do not wrap round to row 0."""
    assert run_host_program(tmp_path, "pixel_coordinates") == ["ok", "65532", "4095"]
