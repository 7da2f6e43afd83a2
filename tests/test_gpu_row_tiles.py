"""The few-row kernel on more than 64 rows: the edges of its tiles of 64 rows and 16, 32 and 64 columns, every way its E8M0 bytes
and words travel (K in chunks, in dwords, in pairs, in single bytes), a C with a frame around it, and NaN blocks that must stay in their
rows and columns.  K past 1024 is what the dispatcher takes: in chunks (4096), in dwords (2560, 7680), in pairs with one chunk (1088) and two
(5184), in single bytes with one (1056) and two (5152), and whole chunks whose arrays start on even and odd addresses (2048)."""
import numpy as np
import pytest

from test_gpu_row_pieces import close, dev, mx, operand, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N", [(65, 1), (127, 31), (128, 64), (193, 130)])
@pytest.mark.parametrize("K,shift", [(512, 0), (544, 0), (1088, 0), (2560, 0), (4096, 0), (7680, 0), (1056, 0), (5152, 0), (5184, 0), (2048, 2), (2048, 1),
                                     (4608, 1)])
def test_row_tiles(mx, oracle, M, N, K, shift):  # noqa: F811
    """shift: scale and word arrays that start 0, 2 or 1 bytes past a 16-byte boundary."""
    rng = np.random.default_rng(M + K)
    a, b = operand(rng, M, K), operand(rng, N, K)
    a[1][[3, M - 1], 0] = 255
    nan = np.zeros((M, N), bool)
    nan[[3, M - 1]] = True
    if N > 1:  # (a single column stays a number: its values are compared)
        b[1][N // 2, K // 32 - 1] = 255
        nan[:, N // 2] = True
    da, db = [dev(a[0])] + [dev(t, shift) for t in a[1:]], [dev(b[0])] + [dev(t, shift) for t in b[1:]]
    for am, bm in ((True, True), (False, False), (True, False)):
        want = oracle.gemm((a[0], a[1], a[2] if am else None), (b[0], b[1], b[2] if bm else None))
        args = (da[0], da[1], da[2] if am else None, db[0], db[1], db[2] if bm else None)
        got = [mx.mx_gemm_mbs(*args, "f32")]  # (what these sizes take)
        for shape in (17, 18, 19):
            if (shape >= 18 and (K % 64 or shift % 2)) or (shape == 19 and (K % 512 or shift)):
                continue
            big = torch.full((M + 1, N + 3), -3.0, device="cuda")
            with mx.forced(gemm_shape=shape):
                mx.mx_gemm_mbs(*args, "f32", out=big[:M, 1:N + 1])
                half = mx.mx_gemm_mbs(*args, "bf16")
            got.append(big[:M, 1:N + 1].clone())
            big[:M, 1:N + 1] = -3.0
            assert bool((big == -3.0).all()), shape
            assert torch.equal(half.nan_to_num(), got[-1].to(torch.bfloat16).nan_to_num()), shape
        for g in got:
            g = g.cpu().numpy()
            assert np.array_equal(np.isnan(g), nan), (K, am, bm)
            close(g[~nan], want[~nan], (K, am, bm))
