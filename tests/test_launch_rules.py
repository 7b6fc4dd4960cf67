"""The GPU tests of kernels with several launch shapes name the shape each of their cases is to run: checked
here against the rules of the library's header, so that a rule that moves cannot leave a shape
untested.  And the rule of the single kernel's groups at sizes where it was measured."""
import pytest

import test_gpu_backward_stages as backward_stages
import test_gpu_contract_edges as contract_edges
import test_gpu_flex_calibrate as flex_calibrate
import test_gpu_fp32_contract as fp32_contract
import test_gpu_fused_small as fused_small
from test_host_indexing import needs_hipcc, run_host_program

pytestmark = needs_hipcc


def rules(tmp_path, layers):
    """(contract_tile_rows, fused_tiles, f32_contract_blocks and backward_from_registers as numbers of two
    digits) of each (m, N, H, W, C, K, bits)."""
    args = [str(v) for layer in layers for v in layer]
    out = [int(v) for v in run_host_program(tmp_path, "launch_rules", args)]
    assert len(out) == 4 * len(layers)
    return list(zip(out[::4], out[1::4], out[2::4], out[3::4]))


def test_contraction_cases_run_the_block_they_name(tmp_path):
    got = rules(tmp_path, [(4, *shape, 8) for shape, _ in contract_edges.CASES])
    assert [g[0] for g in got] == [rows for _, rows in contract_edges.CASES]
    assert {g[0] for g in got} == {64, 128}


def test_flex_calibration_cases_run_the_block_they_name(tmp_path):
    cases = flex_calibrate.WIDE_CASES
    got = rules(tmp_path, [(m, *shape, 8) for m, _, _, _, _, shape in cases])
    assert [g[0] for g in got] == [128] * len(cases)


def test_single_kernel_cases_run_the_group_they_name(tmp_path):
    cases = fused_small.CASES
    got = rules(tmp_path, [(c[0], *c[6], c[2]) for c in cases])
    assert [g[1] for g in got] == [c[7] for c in cases]
    sixteen = [c for c in cases if c[7] == 16]
    assert {c[0] for c in sixteen} == {2, 4} and {c[2] for c in sixteen} == {8, 9}
    assert {c[5] for c in sixteen} == {True, False} and {c[1] for c in sixteen} == {"canonical", "legendre"}


def test_fp32_contraction_cases_run_the_blocks_they_name(tmp_path):
    got = rules(tmp_path, [(*c[:6], 8) for c in fp32_contract.CASES])
    assert [g[2] for g in got] == [c[6] for c in fp32_contract.CASES]
    assert {g[2] for g in got} == {11, 12, 21, 22}


def test_backward_cases_run_the_bodies_they_name(tmp_path):
    got = rules(tmp_path, [(4, *shape, 8) for shape, _ in backward_stages.CASES])
    assert [g[3] for g in got] == [registers for _, registers in backward_stages.CASES]
    by_tile = {(shape[4] > 64, shape[3] > 64, registers) for shape, registers in backward_stages.CASES}
    assert len(by_tile) == 12         # every tile shape with every choice


@pytest.mark.parametrize("m,T,K,bits,tiles", [
    (4, 1024, 64, 8, 4), (4, 4096, 64, 8, 8), (4, 8192, 64, 8, 16), (4, 10240, 64, 8, 8),
    (2, 9216, 64, 8, 16), (2, 10240, 64, 8, 16),       # 11.8 us against 12.4 with 8 tiles
    (2, 10240, 16, 8, 8), (2, 10240, 48, 8, 8), (2, 4096, 64, 8, 8), (2, 5120, 64, 9, 8), (4, 4096, 64, 9, 16),
])
def test_single_kernel_group_where_it_was_measured(tmp_path, m, T, K, bits, tiles):
    assert rules(tmp_path, [(m, T, m, m, 64, K, bits)])[0][1] == tiles
