"""The 8-bit and 6-bit GEMM on 64 x 128 tiles, where they can go wrong: the edges of a tile, K's last group of four stages whole,
one block pair long and one short, rows of scales at any address, groups that end inside a tile.  The tile shapes and the
general form add the same products in the same order: their results are the same bits.  The tiles themselves are held to the oracle too."""
import numpy as np
import pytest

from test_gpu_parity_elem import ALL_PAIRS, assert_gemm_elem_ok, gpu_gemm, random_operand_any
from test_gpu_row_pieces import dev, mx, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def operand(mx, rng, rows, K, elem):  # noqa: F811
    return (rng.integers(0, 120, (rows, mx.elem_code_bytes(elem, K)), dtype=np.uint8), rng.integers(120, 130, (rows, K // 32), dtype=np.uint8),
            rng.integers(0, 256, (rows, (K + 127) // 128), dtype=np.uint8))


@pytest.mark.parametrize("elem", ["e4m3", "e3m2"])
@pytest.mark.parametrize("M,N,K", [(1, 127, 512), (63, 129, 576), (64, 128, 960), (65, 1, 1024), (130, 257, 1600), (300, 140, 2880)])
def test_tiles_agree(mx, elem, M, N, K):  # noqa: F811
    rng = np.random.default_rng(M + N + K)
    a, b = operand(mx, rng, M, K, elem), operand(mx, rng, N, K, elem)
    da, db = [dev(a[0])] + [dev(t, 2) for t in a[1:]], [dev(b[0])] + [dev(t, 2) for t in b[1:]]
    if K % 128 == 0:  # (whole macro blocks want dword-aligned E8M0 bytes)
        da[1], db[1] = dev(a[1]), dev(b[1])
    for words in (True, False):
        got = []
        for force in (1, 16, 17, 18):
            with mx.forced(gemm_elem=force):
                got.append(mx.mx_gemm_mbs_elem(elem, da[0], da[1], da[2] if words else None, elem, db[0], db[1], db[2] if words else None, "f32"))
        assert all(torch.equal(g, got[0]) for g in got), (elem, words)


@pytest.mark.parametrize("elem", ["e5m2", "e2m3"])
def test_groups_of_few_rows(mx, elem):  # noqa: F811
    rng = np.random.default_rng(7)
    sizes = [0, 1, 64, 65, 0, 130, 7]
    M, N, K = sum(sizes), 200, 1088
    a, w = operand(mx, rng, M, K, elem), operand(mx, rng, len(sizes) * N, K, elem)
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(sizes)]), device="cuda")
    da, dw = [dev(t) for t in a], [dev(t) for t in w]
    got = mx.mx_gemm_mbs_elem_grouped(elem, *da, elem, *dw, offsets, N, "f32")
    for e in range(len(sizes)):
        lo, hi = int(offsets[e]), int(offsets[e + 1])
        if lo < hi:
            with mx.forced(gemm_elem=16):
                want = mx.mx_gemm_mbs_elem(elem, *[t[lo:hi].contiguous() for t in da], elem, *[t[e * N:(e + 1) * N].contiguous() for t in dw], "f32")
            assert torch.equal(got[lo:hi], want), (elem, e)


# (one group of four stages whole, a group of one block pair, three stages, several groups with a short one; with words on both sides, one, none)
@pytest.mark.parametrize("ea,eb", ALL_PAIRS)
def test_against_the_oracle(mx, oracle, ea, eb):  # noqa: F811
    rng = np.random.default_rng(64)
    hi = 132 if "e5m2" in (ea, eb) else 140
    for M, N, K in ((63, 129, 512), (65, 40, 576), (130, 131, 896), (33, 257, 2880)):
        (a, pa), (b, pb) = random_operand_any(rng, ea, M, K, 110, hi), random_operand_any(rng, eb, N, K, 110, hi)
        for wa, wb in ((True, True), (False, True), (False, False)):
            got = gpu_gemm(mx, ea, (pa[0], pa[1], pa[2] if wa else None), eb, (pb[0], pb[1], pb[2] if wb else None), kernel=18)
            assert_gemm_elem_ok(oracle, got.cpu().numpy(), ea, (a[0], a[1], a[2] if wa else None), eb, (b[0], b[1], b[2] if wb else None),
                                "64 x 128 tiles %s x %s %dx%dx%d words %d%d" % (ea, eb, M, N, K, wa, wb))
