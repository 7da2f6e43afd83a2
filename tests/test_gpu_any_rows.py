"""The main GEMM kernel's general form (a row's E8M0 bytes and MBS words as pieces through registers) where K ends in one or
three blocks of a macro block or the arrays sit on odd addresses: K's last group of four macro blocks whole, one block long, one
block short and alone; a NaN block at the start of the rows behind a partial group, which must not reach the rows before them."""
import numpy as np
import pytest

from test_gpu_row_pieces import close, dev, mx, operand, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [None, 8, 9, 12])
@pytest.mark.parametrize("K,shift", [(32, 0), (96, 1), (416, 0), (480, 3), (512, 1), (544, 0), (608, 1), (992, 0), (1024, 1), (2080, 0), (2144, 1)])
def test_odd_blocks_and_addresses(mx, oracle, shape, K, shift):  # noqa: F811
    rng = np.random.default_rng(K)
    M, N = 261, 139
    a, b = operand(rng, M, K), operand(rng, N, K)
    a[1][[3, 260], 0] = 255
    b[1][[1, 138], 0] = 255
    da, db = [dev(a[0])] + [dev(t, shift) for t in a[1:]], [dev(b[0])] + [dev(t, shift) for t in b[1:]]
    nan = np.zeros((M, N), bool)
    nan[[3, 260]] = True
    nan[:, [1, 138]] = True
    for am, bm in ((True, True), (False, False), (False, True)):
        if shape == 12 and not (am or bm):
            continue
        want = oracle.gemm((a[0], a[1], a[2] if am else None), (b[0], b[1], b[2] if bm else None))
        args = (da[0], da[1], da[2] if am else None, db[0], db[1], db[2] if bm else None, "f32")
        if shape is None:
            got = mx.mx_gemm_mbs(*args)
        else:
            with mx.forced(gemm_shape=shape):
                got = mx.mx_gemm_mbs(*args)
        got = got.cpu().numpy()
        assert np.array_equal(np.isnan(got), nan), (K, am, bm)
        close(got[~nan], want[~nan], (K, am, bm))
    # grouped: the second group's rows and weight start behind a partial row of the first
    offsets = torch.tensor([0, 100, 100, M], device="cuda")
    w = operand(rng, 3 * N, K)
    got = mx.mx_gemm_mbs_grouped(*da, *[dev(w[0])] + [dev(t, shift) for t in w[1:]], offsets, N, "f32").cpu().numpy()
    for e, (lo, hi) in enumerate(((0, 100), (100, 100), (100, M))):
        rows = [r for r in range(lo, hi) if r not in (3, 260)]
        if rows:
            want = oracle.gemm(tuple(t[rows] for t in a), tuple(t[e * N:(e + 1) * N] for t in w))
            close(got[rows], want, (K, "group", e))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N", [(1, 1), (5, 130), (261, 139), (3, 4096)])
def test_empty_sum(mx, dtype, M, N):  # noqa: F811
    """K = 0: zeros in C's rows and nothing beside them; grouped, in the rows that belong to a group."""
    empty = lambda rows: [torch.empty((rows, 0), dtype=torch.uint8, device="cuda") for _ in range(3)]  # noqa: E731
    full = torch.full((M + 2, N + 3), -3.0, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
    offsets = torch.tensor([0, 0, M // 2, M - M // 3], device="cuda")
    for call, rows in ((lambda out: mx.mx_gemm(*empty(M)[:2], *empty(N)[:2], dtype, out=out), M), (lambda out: mx.mx_gemm_mbs(*empty(M), *empty(N), dtype, out=out), M),
                       (lambda out: mx.mx_gemm_mbs_grouped(*empty(M), *empty(3 * N), offsets, N, dtype, out=out), M - M // 3)):
        big = full.clone()
        call(big[1:M + 1, 1:N + 1])
        want = full.clone()
        want[1:rows + 1, 1:N + 1] = 0
        assert torch.equal(big, want)
    assert mx.gemm_plan(M, N, 0) == "gemm_zero_kernel"
