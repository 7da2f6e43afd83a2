"""Outputs of more than one round of 64 x 128 tiles, where the tile shape is chosen by what each kernel takes: short and long K, whole and
part rounds, so that each shape is chosen somewhere.  All shapes, which other tests hold to the oracle, give the same bits."""
import numpy as np
import pytest

from test_gpu_row_pieces import mx, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def operand(mx, seed, rows, K, elem=None):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda cols, lo, hi: torch.randint(lo, hi, (rows, cols), generator=g, device="cuda", dtype=torch.uint8)  # noqa: E731
    return r(mx.elem_code_bytes(elem, K), 0, 120) if elem else r(K // 2, 0, 256), r(K // 32, 120, 130), r((K + 127) // 128, 0, 256)


@pytest.mark.parametrize("M,N,K", [(2067, 1031, 512), (1579, 2784, 1024), (716, 2786, 1536), (300, 9001, 576), (2051, 1160, 1632), (1031, 4099, 96)])
def test_four_bit(mx, M, N, K):  # noqa: F811
    a, b = operand(mx, 1, M, K), operand(mx, 2, N, K)
    for words, fast in ((True, (3, 4, 11)), (False, (2, 6, 7))):
        call = lambda: mx.mx_gemm_mbs(*a, *b, "f32") if words else mx.mx_gemm(*a[:2], *b[:2], "f32")  # noqa: E731
        want = call()
        for shape in (fast if K % 512 == 0 else ()) + ((8, 9, 12) if words else (8, 9)):
            with mx.forced(gemm_shape=shape):
                assert torch.equal(call(), want), (words, shape)


@pytest.mark.parametrize("elem", ["e4m3", "e3m2"])
@pytest.mark.parametrize("M,N,K", [(784, 6290, 512), (716, 2786, 576), (2594, 1121, 960), (300, 11471, 1024)])
def test_eight_and_six_bit(mx, elem, M, N, K):  # noqa: F811
    a, b = operand(mx, 1, M, K, elem), operand(mx, 2, N, K, elem)
    for words in (True, False):
        call = lambda: mx.mx_gemm_mbs_elem(elem, a[0], a[1], a[2] if words else None, elem, b[0], b[1], b[2] if words else None, "f32")  # noqa: E731
        want = call()
        for force in (1, 16, 17, 18):
            with mx.forced(gemm_elem=force):
                assert torch.equal(call(), want), (words, force)
