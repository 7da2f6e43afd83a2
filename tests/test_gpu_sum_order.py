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
