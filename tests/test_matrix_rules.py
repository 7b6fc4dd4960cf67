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
    # one group per compute unit, and one more (9 bits: two blocks of channels)
    lines = [(1, 128, 128, 64, 8), (1, 128, 129, 64, 8), (2, 128, 128, 64, 8), (33, 4, 252, 64, 8),
             (2, 64, 64, 64, 9), (2, 64, 65, 64, 9), (4, 64, 64, 64, 9), (4, 64, 65, 64, 9)]
    got = run_host_program(tmp_path, "matrix_rules", [str(v) for line in lines for v in line])
    assert [int(v) for v in got] == [4, 8, 8, 16, 4, 8, 8, 16]


def test_dealing_of_block_pairs(tmp_path):
    assert run_host_program(tmp_path, "pair_dealing")[0] == "ok"


def test_sixteen_bit_pixel_coordinates(tmp_path):
    """Tiles reach past the image: 65532 rows are the most whose padding rows do not wrap round to row 0."""
    assert run_host_program(tmp_path, "pixel_coordinates") == ["ok", "65532", "4095"]


# N, H, W, C, K: routes of input alone, input beside filters, output to fp32, output to int8 (int8 M)
INPUT_LINES = [((1535, 8, 8, 16, 16), "0011"), ((1536, 8, 8, 16, 16), "1111"),      # 3 * 2^15 items
               ((511, 4, 4, 512, 512), "1011"), ((1024, 4, 4, 512, 512), "1101"),   # twice the filters
               ((1023, 4, 4, 512, 512), "1001")]
OUTPUT_LINES = [((1536, 8, 8, 64, 64), "1111"), ((1537, 8, 8, 64, 64), "1101"),      # 3 * 2^17 items
                ((4095, 8, 8, 64, 64), "1101"), ((4096, 8, 8, 64, 64), "1111"),      # 2^20
                ((8192, 8, 8, 64, 64), "1101"), ((2048, 8, 8, 256, 256), "1100"),    # 2^21: planes 2 MiB apart
                ((2049, 8, 8, 256, 256), "1101"),                                    # whole tiles
                ((4096, 16, 16, 85 * 16, 16), "1111"), ((4096, 16, 16, 96, 96), "1100")]  # more than 192 MB of M


def routes(tmp_path, layers):
    return run_host_program(tmp_path, "matrix_routes", [str(v) for layer in layers for v in layer])


def test_lines_between_vector_and_matrix_form(tmp_path):
    lines = INPUT_LINES + OUTPUT_LINES
    assert routes(tmp_path, [layer for layer, _ in lines]) == [want for _, want in lines]


def test_input_cases_run_on_the_matrix_pipe(tmp_path):
    got = routes(tmp_path, [(*shape, 16) for shape in brackets.MATRIX_INPUTS])
    assert all(r.startswith("11") for r in got)
