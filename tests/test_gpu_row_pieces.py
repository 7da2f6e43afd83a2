"""GEMMs whose rows of E8M0 bytes and MBS words start anywhere, at the K where the pieces they are fetched in change:
K's last group of four macro blocks whole, one pair of blocks long, one pair short, and alone; a NaN block at the start of
the rows behind a partial group, which must not reach the rows before them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_08713_amd as mx_

    mx_.load_library()
    return mx_


def dev(a, shift=0):
    """On the GPU, `shift` bytes into an allocation (rows stay contiguous)."""
    flat = torch.zeros(a.size + shift, dtype=torch.uint8, device="cuda")
    flat[shift:] = torch.from_numpy(a.reshape(-1)).cuda()
    return flat[shift:].view(a.shape)


def operand(rng, rows, K):
    return (rng.integers(0, 256, (rows, K // 2), dtype=np.uint8), rng.integers(110, 140, (rows, K // 32), dtype=np.uint8),
            rng.integers(0, 256, (rows, (K + 127) // 128), dtype=np.uint8))


def close(got, want, what):
    # 1e-3 of the RMS is the interface's bound on the fp32 output
    err, rms = np.nanmax(np.abs(got.astype(np.float64) - want)), np.sqrt(np.nanmean(want ** 2))
    assert err <= 1e-3 * rms, (what, err, rms)


# (shape 8, 9, 12: 256 x 128, 128 x 128 and, with words only, 64 x 128 tiles)
@pytest.mark.parametrize("shape", [8, 9, 12])
@pytest.mark.parametrize("K,shift", [(64, 0), (448, 2), (512, 2), (576, 0), (960, 0), (1024, 2), (1088, 2), (1984, 0), (2880, 2)])
def test_mxfp4(mx, oracle, shape, K, shift):
    rng = np.random.default_rng(K + shape)
    M, N = 261, 139
    a, b = operand(rng, M, K), operand(rng, N, K)
    a[1][[3, 260], 0] = 255
    b[1][[1, 138], 0] = 255
    da, db = [dev(a[0])] + [dev(t, shift) for t in a[1:]], [dev(b[0])] + [dev(t, shift) for t in b[1:]]
    nan = np.zeros((M, N), bool)
    nan[[3, 260]] = True
    nan[:, [1, 138]] = True
    with mx.forced(gemm_shape=shape):
        for am, bm in ((True, True), (False, False), (True, False)):
            if shape == 12 and not (am or bm):
                continue
            want = oracle.gemm((a[0], a[1], a[2] if am else None), (b[0], b[1], b[2] if bm else None))
            got = mx.mx_gemm_mbs(da[0], da[1], da[2] if am else None, db[0], db[1], db[2] if bm else None, "f32").cpu().numpy()
            assert np.array_equal(np.isnan(got), nan), (K, am, bm)
            close(got[~nan], want[~nan], (K, am, bm))


@pytest.mark.parametrize("K", [64, 128, 192, 256, 320, 384, 448])
def test_mxfp4_short_rows(mx, oracle, K):
    """Rows of fewer than 16 E8M0 bytes, one of every length, that start on every second even address; a NaN block in the first
    and in the last place of a row."""
    rng = np.random.default_rng(K)
    M, N = 133, 129
    a, b = operand(rng, M, K), operand(rng, N, K)
    a[1][3, -1] = a[1][132, 0] = b[1][1, 0] = b[1][128, -1] = 255
    nan = np.zeros((M, N), bool)
    nan[[3, 132]] = True
    nan[:, [1, 128]] = True
    da, db = [dev(a[0])] + [dev(t, 2) for t in a[1:]], [dev(b[0])] + [dev(t, 2) for t in b[1:]]
    for shape in (8, 9, 12):
        for mbs in (True, False):
            if shape == 12 and not mbs:
                continue
            with mx.forced(gemm_shape=shape):
                got = mx.mx_gemm_mbs(da[0], da[1], da[2] if mbs else None, db[0], db[1], db[2] if mbs else None, "f32").cpu().numpy()
            want = oracle.gemm((a[0], a[1], a[2] if mbs else None), (b[0], b[1], b[2] if mbs else None))
            assert np.array_equal(np.isnan(got), nan), (shape, mbs)
            close(got[~nan], want[~nan], (K, shape, mbs))


@pytest.mark.parametrize("M,N,K", [(65, 130, 512), (64, 128, 1024), (193, 300, 1536), (129, 4097, 2560)])
def test_mxfp4_64_row_tiles(mx, oracle, M, N, K):
    """The 64 x 128 tile of the fast form, which few tiles take: against the oracle, bit for bit the 128 x 128 tile's result,
    and C's neighbours untouched."""
    rng = np.random.default_rng(M + K)
    a, b = operand(rng, M, K), operand(rng, N, K)
    da, db = [dev(t) for t in a], [dev(t) for t in b]
    got = {}
    for shape in (11, 4):
        with mx.forced(gemm_shape=shape):
            big = torch.full((M + 2, N + 3), -3.0, dtype=torch.float32, device="cuda")
            mx.mx_gemm_mbs(*da, *db, "f32", out=big[1:M + 1, 1:N + 1])
            got[shape] = big[1:M + 1, 1:N + 1].clone()
            big[1:M + 1, 1:N + 1] = -3.0
            assert bool((big == -3.0).all())
    assert torch.equal(got[11], got[4])
    close(got[11].cpu().numpy(), oracle.gemm(a, b), (M, N, K))
