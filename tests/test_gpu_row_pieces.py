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


# (shape 8, 9: 256 x 128 and 128 x 128 tiles)
@pytest.mark.parametrize("shape", [8, 9])
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
            want = oracle.gemm((a[0], a[1], a[2] if am else None), (b[0], b[1], b[2] if bm else None))
            got = mx.mx_gemm_mbs(da[0], da[1], da[2] if am else None, db[0], db[1], db[2] if bm else None, "f32").cpu().numpy()
            assert np.array_equal(np.isnan(got), nan), (K, am, bm)
            close(got[~nan], want[~nan], (K, am, bm))
