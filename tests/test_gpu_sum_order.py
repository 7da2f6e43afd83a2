"""Calls of few rows whose sum over K the few-row kernel splits over its wavefronts, with a smaller error than the tiles' single chain:
the dispatcher leaves them there, and the error against 64-bit arithmetic says so."""
import pytest

from test_gpu_row_pieces import mx, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def quantized(mx, seed, rows, K, elem=None, scale=1.0):  # noqa: F811
    x = (torch.randn((rows, K), generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda") * scale).to(torch.bfloat16)
    return mx.mx_quantize_mbs(x, "oas") if elem is None else mx.mx_quantize_elem(x, elem)


def value(mx, q, elem=None):  # noqa: F811
    plain = mx.mx_dequantize(q[0], q[1], None, "f32") if elem is None else mx.mx_dequantize_elem(elem, q[0], q[1], None, "f32")
    return plain.double() / (1 + q[2].double() / 256).repeat_interleave(128, 1)[:, :plain.shape[1]]


def error(got, want):
    return float((got.double() - want).norm() / want.norm())


@pytest.mark.parametrize("G,rows,N,K", [(8, 16, 2048, 2048), (16, 24, 1056, 2112), (4, 32, 4096, 4096)])
def test_groups(mx, G, rows, N, K):  # noqa: F811
    a, b = quantized(mx, 1, G * rows, K), quantized(mx, 2, G * N, K, scale=0.02)
    offsets = torch.arange(0, G * rows + 1, rows, device="cuda")
    call = lambda: mx.mx_gemm_mbs_grouped(*a, *b, offsets, N, "f32")  # noqa: E731
    got = call()
    with mx.forced(gemm_shape=5):
        few = call()
    with mx.forced(gemm_shape=12):
        tiles = call()
    x, w = value(mx, a), value(mx, b)
    want = torch.cat([x[e * rows:(e + 1) * rows] @ w[e * N:(e + 1) * N].T.contiguous() for e in range(G)])
    assert torch.equal(got, few)
    assert error(got, want) < error(tiles, want) < 2e-7


@pytest.mark.parametrize("M,N,K", [(32, 33556, 1824), (2, 50884, 2592)])
def test_single_scale_bytes(mx, M, N, K):  # noqa: F811
    """K % 64 = 32 in several rounds of workgroups."""
    a, b = quantized(mx, 1, M, K), quantized(mx, 2, N, K, scale=0.02)
    got = mx.mx_gemm_mbs(*a, *b, "f32")
    with mx.forced(gemm_shape=5):
        few = mx.mx_gemm_mbs(*a, *b, "f32")
    with mx.forced(gemm_shape=12):
        tiles = mx.mx_gemm_mbs(*a, *b, "f32")
    want = value(mx, a) @ value(mx, b).T.contiguous()
    assert torch.equal(got, few)
    assert error(got, want) < error(tiles, want) < 2e-7


@pytest.mark.parametrize("a_elem,b_elem,M,N,K", [("e2m3", "e2m3", 64, 4224, 1024), ("e2m3", "e3m2", 33, 8200, 2048), ("e3m2", "e2m3", 8, 16896, 4096)])
def test_e2m3(mx, a_elem, b_elem, M, N, K):  # noqa: F811
    """E2M3 on either side: its products are exact in the matrix unit, so the order of the sum over K decides the error."""
    a, b = quantized(mx, 1, M, K, a_elem), quantized(mx, 2, N, K, b_elem, scale=0.02)
    call = lambda: mx.mx_gemm_mbs_elem(a_elem, *a, b_elem, *b, "f32")  # noqa: E731
    got = call()
    with mx.forced(gemm_elem=3):
        few = call()
    with mx.forced(gemm_elem=18):
        tiles = call()
    want = value(mx, a, a_elem) @ value(mx, b, b_elem).T.contiguous()
    assert torch.equal(got, few)
    assert error(got, want) < error(tiles, want) < 2e-7


# (rounds of 4096 columns: four and five; more than 32 rows in one round: short and long K, with words and without)
@pytest.mark.parametrize("elem,words,M,N,K,few", [("e4m3", True, 8, 16384, 4096, True), ("e4m3", True, 8, 16500, 4096, False), ("e5m2", True, 40, 300, 1024, True),
                                                  ("e4m3", True, 64, 300, 1536, True), ("e4m3", True, 64, 300, 1024, False), ("e4m3", False, 33, 300, 3072, True),
                                                  ("e4m3", False, 41, 300, 3072, False), ("e4m3", False, 12, 16400, 8192, False), ("e2m3", True, 41, 4100, 1024, True),
                                                  ("e2m3", False, 41, 4100, 1024, False),
                                                  ("e4m3", True, 56, 300, 1024, True), ("e3m2", True, 64, 4096, 1024, True),
                                                  ("e3m2", False, 8, 16384, 1024, True), ("e3m2", False, 9, 16384, 512, True), ("e3m2", False, 9, 8200, 1024, False),
                                                  ("e3m2", False, 8, 16385, 512, False), ("e3m2", False, 8, 8200, 1536, False), ("e4m3", False, 8, 8200, 1024, False)])
def test_lines_of_the_few_row_kernel(mx, elem, words, M, N, K, few):  # noqa: F811
    """Which kernel 8-bit and 6-bit calls take, by the sums' bits: the few-row kernel's, or the tiles', which differ on such operands."""
    a, b = quantized(mx, 1, M, K, elem), quantized(mx, 2, N, K, elem, 0.02)
    if not words:  # (what is exact in every order says nothing: scales far apart)
        a[1].copy_(torch.randint(100, 150, a[1].shape, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda", dtype=torch.uint8))
        b[1].copy_(torch.randint(100, 150, b[1].shape, generator=torch.Generator(device="cuda").manual_seed(4), device="cuda", dtype=torch.uint8))
    got = {}
    for force in (0, 3, 18):
        with mx.forced(gemm_elem=force):
            got[force] = mx.mx_gemm_mbs_elem(elem, a[0], a[1], a[2] if words else None, elem, b[0], b[1], b[2] if words else None, "f32")
    assert torch.equal(got[0], got[3 if few else 18]) and not torch.equal(got[3], got[18])
