"""Sizes that callers allocate by, on the host: a buffer made for a batch has to serve every smaller one."""
import pytest

from paper_2602_05145_amd import binding as B


@pytest.mark.parametrize("d", [8, 256, 1000, 1023, 2048, 2056, 4096, 8192])
def test_rmsnorm_scratch_never_falls_as_rows_grow(d):
    sizes = [B.tide_rmsnorm_bwd_scratch_bytes(rows, d) for rows in range(1, 16500)]
    assert sizes == sorted(sizes)
    assert sizes[0] == 4 * d and sizes[479] >= 480 * 4 * d      # a partial sum per block, a block per row up to 480
    assert sizes[-1] <= 16 << 20                                # the fixed array of tide_rmsnorm_bwd_static
