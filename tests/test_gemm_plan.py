"""Which kernel a problem takes (host code, no GPU): the lines that precision and launch limits draw."""
import pytest

import paper_2603_08713_amd as mx


@pytest.mark.parametrize("G,rows,dim", [(8, 16, 2048), (16, 24, 2112), (32, 32, 2880), (64, 32, 1024), (64, 32, 768), (8, 1, 5120)])
def test_groups_of_few_rows_keep_the_split_sum(G, rows, dim):
    """With more than five macro blocks (seven excepted) the tiles' single chain over K is less exact than the few-row kernel's four shares."""
    assert "few rows per group" in mx.gemm_plan(G * rows, dim, dim, grouped=True, num_groups=G)


def test_groups_of_few_rows_on_tiles():
    assert "64x128" in mx.gemm_plan(64 * 32, 2048, 640, grouped=True, num_groups=64)
    assert "64x128" in mx.gemm_plan(64 * 32, 2048, 896, grouped=True, num_groups=64)
    assert "few rows" in mx.gemm_plan(64 * 32, 2048, 672, grouped=True, num_groups=64)
