"""The MBS-Dynamic search takes listed words four at a time, lists of up to seven words and of nine one at a time: lists of every length about a multiple of four, with the static
word among the candidates (listed once) and not (listed in front of them), on whole and ragged rows."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from test_gpu_parity import assert_dynamic_valid  # noqa: E402


@pytest.fixture(scope="module")
def mx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_08713_amd as mx_

    mx_.load_library()
    return mx_


@pytest.mark.parametrize("first", [0, 1, -7])
@pytest.mark.parametrize("count", [1, 2, 3, 4, 5, 8, 9])
def test_list_lengths(mx, oracle, first, count):
    from paper_2603_08713_amd import synth

    bits = synth.activations_student_t(9, 512 + 160, 3.0, 0.01, 50.0, 100 + count)
    for rule in ("oas", "ocp"):
        assert_dynamic_valid(mx, oracle, bits, rule, "list", cand_first=first, cand_count=count, cand_stride=16)
