"""The rules of the library's header that choose launch shapes, at sizes where they were measured."""
import pytest

from test_host_indexing import needs_hipcc, run_host_program

pytestmark = needs_hipcc


def rules(tmp_path, layers):
    """(contract_tile_rows, fused_tiles) of each (m, N, H, W, C, K, bits)."""
    args = [str(v) for layer in layers for v in layer]
    out = [int(v) for v in run_host_program(tmp_path, "launch_rules", args)]
    assert len(out) == 2 * len(layers)
    return list(zip(out[::2], out[1::2]))


@pytest.mark.parametrize("m,T,K,bits,tiles", [
    (4, 1024, 64, 8, 4), (4, 4096, 64, 8, 8), (4, 8192, 64, 8, 16), (4, 10240, 64, 8, 8),
    (2, 9216, 64, 8, 16), (2, 10240, 64, 8, 16),       # 11.8 us against 12.4 with 8 tiles
    (2, 10240, 16, 8, 8), (2, 10240, 48, 8, 8), (2, 4096, 64, 8, 8), (2, 5120, 64, 9, 8), (4, 4096, 64, 9, 16),
])
def test_single_kernel_group_where_it_was_measured(tmp_path, m, T, K, bits, tiles):
    assert rules(tmp_path, [(m, T, m, m, 64, K, bits)])[0][1] == tiles
