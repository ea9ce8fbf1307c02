"""The selector's workgroups: as many as row tiles of 64 rows of a chunk give units, the CUs at most."""
import pytest

from paper_2601_06562_amd import binding


@pytest.mark.parametrize("rows,d,V,budget,cus", [(1, 64, 300, 0, 0), (32, 64, 8192, 0, 0), (33, 512, 8192, 0, 0), (268, 512, 8192, 0, 0),
                                                 (268, 512, 8192, 0, 64), (512, 512, 8192, 7000, 0), (4096, 4096, 126464, 0, 0),
                                                 (300, 1024, 32000, 20000, 0), (2000, 64, 256, 0, 0)])
def test_workgroups_of_a_plan(rows, d, V, budget, cus):
    p = binding.mosaic_plan_workspace(4096, rows, d, V, budget, cus)
    K = next(k for k in range(1, rows + 1) if -(-(-(-rows // k)) // 256) * 256 == p.rows_per_chunk)
    units = -(-(-(-rows // K)) // 64) * p.vocab_splits
    assert p.grid == min(units, cus or 256)
