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


@pytest.mark.parametrize("M,N,K,a,b", [(32, 33556, 1824, 1, 1), (2, 50884, 2592, 1, 1), (27, 12681, 1312, 1, 1), (5, 33505, 1184, 1, 0), (16, 56399, 5152, 1, 0), (8, 20000, 1696, 0, 0),
                                       (45, 5264, 352, 1, 0), (25, 6218, 480, 0, 0)])
def test_single_bytes_stay_on_the_few_row_kernel(M, N, K, a, b):
    """K % 64 = 32: past K = 1024 the split sum is the more exact one; below, where tiles take longer."""
    assert "few rows" in mx.gemm_plan(M, N, K, bool(a), bool(b))


def test_single_bytes_on_tiles():
    assert "few rows" not in mx.gemm_plan(56, 14000, 864) and "few rows" not in mx.gemm_plan(64, 28672, 4128)


def test_tiles_whose_grid_a_launch_takes():
    """Twice as many work-items as on 256 x 128 tiles: from 2^32 on the launch would be refused."""
    assert "256x128" in mx.gemm_plan(300 * 3300000, 100, 32, grouped=True, num_groups=3300000)
    assert "64x128" in mx.gemm_plan(300 * 33000, 100, 32, grouped=True, num_groups=33000)


@pytest.mark.parametrize("M,N,K,tile", [(4826, 15920, 1024, "256x256"), (7130, 11368, 1024, "256x256"), (2939, 8592, 1024, "256x256"), (3000, 3000, 4096, "256x256"),
                                        (4826, 15917, 1024, "128x128"), (718, 11043, 8192, "256x256"),
                                        (4096, 14336, 512, "128x128"), (4096, 14344, 512, "128x128"),
                                        (3498, 3584, 1024, "128x128"), (4096, 14336, 1536, "128x128"), (3498, 3584, 2048, "256x256")])
def test_plain_tiles_by_the_rows_of_c(M, N, K, tile):
    """Without words: by price as long as K is short, longest where rows of C start on any element, shortest where they start on 16 bytes; else by area."""
    assert tile in mx.gemm_plan(M, N, K, False, False)


@pytest.mark.parametrize("M,N,K,tile", [(784, 6272, 512, "256x128"), (784, 6280, 512, "64x128"), (1500, 2048, 576, "128x128"), (1500, 2048, 1984, "128x128"), (1500, 2048, 7744, "64x128"),
                                        (1024, 2048, 576, "64x128"), (1300, 2500, 1088, "64x128"), (1300, 2496, 1088, "128x128"), (1024, 8192, 1088, "256x128")])
def test_tiles_for_rows_of_c_on_lines(M, N, K, tile):
    """With words: near a tie of the prices, rows of C on whole lines go to the larger tile."""
    assert " " + tile in mx.gemm_plan(M, N, K)
