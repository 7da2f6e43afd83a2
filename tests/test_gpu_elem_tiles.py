"""GEMMs on 8-bit and 6-bit operands at the edges of the 128 x 128 tile (few tiles) and of the 256 x 128 tile, with K that
fills its last group of four macro blocks, ends one stage or half a stage into it, and takes one turn of the loop and a rest:
the general form multiplies and folds in the same order, so the bits must agree; one shape against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from test_gpu_parity_elem import assert_gemm_elem_ok, gpu_gemm, host, random_operand_any  # noqa: E402


@pytest.fixture(scope="module")
def mx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_08713_amd as mx_

    mx_.load_library()
    return mx_


# 128 x 128 tiles but for the last pair, whose 256 x 128 tiles fill whole rounds
@pytest.mark.parametrize("M,N", [(65, 1), (127, 130), (129, 257), (300, 128), (2048, 4096)])
@pytest.mark.parametrize("K", [512, 576, 640, 1088, 1536, 1600, 2112])
@pytest.mark.parametrize("ea,eb", [("e4m3", "e5m2"), ("e2m3", "e3m2")])
def test_tiles_equal_general_form(mx, oracle, M, N, K, ea, eb):
    if M * N > 1 << 20 and K not in (576, 1536):
        pytest.skip("one partial and one whole K at the large shape")
    rng = np.random.default_rng(M + K)
    (a, pa), (b, pb) = random_operand_any(rng, ea, M, K, 112, 132), random_operand_any(rng, eb, N, K, 112, 132)
    for wa, wb in ((True, True), (False, False), (False, True)):
        p = [(x[0], x[1], x[2] if w else None) for x, w in ((pa, wa), (pb, wb))]
        got = gpu_gemm(mx, ea, p[0], eb, p[1], kernel=2)
        assert torch.equal(got, gpu_gemm(mx, ea, p[0], eb, p[1], kernel=1)), (wa, wb)
        assert torch.equal(gpu_gemm(mx, ea, p[0], eb, p[1], "bf16", kernel=2), got.to(torch.bfloat16)), (wa, wb)
        if (M, N) == (129, 257):
            c = [(x[0], x[1], x[2] if w else None) for x, w in ((a, wa), (b, wb))]
            assert_gemm_elem_ok(oracle, host(got), ea, c[0], eb, c[1], (K, wa, wb))
