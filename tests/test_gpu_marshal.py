"""The binding's native marshaller against its Python path: the same outputs, the same errors, and what it declines."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_08713_amd as mx_

    mx_.load_library()
    mx_.mx_quantize(torch.zeros((1, 32), dtype=torch.bfloat16, device="cuda"))
    assert mx_.binding._native is not None, "the build step makes _marshal.so"
    return mx_


def u8(*shape):
    return torch.empty(shape, dtype=torch.uint8, device="cuda")


def calls(mx):
    """name -> (call with all outputs given, its outputs)"""
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    M, N, K = 33, 96, 512
    x, w = (torch.randn((r, K), generator=g, device="cuda").to(torch.bfloat16) for r in (M, N))
    wide = torch.randn((M, K + 8), generator=g, device="cuda").to(torch.bfloat16)[:, :K]
    q = lambda r, cb=K // 2: (u8(r, cb), u8(r, K // 32), u8(r, K // 128))
    a, b = mx.mx_quantize_mbs(x, "oas"), mx.mx_quantize_mbs(w, "oas")
    ea, eb = mx.mx_quantize_elem(x, "e2m3"), mx.mx_quantize_elem(w, "e3m2")
    big = torch.zeros((M, N + 3), dtype=torch.bfloat16, device="cuda")
    c, f = big[:, 1:N + 1], torch.zeros((M, N), device="cuda")
    half = torch.zeros((M, N // 2), device="cuda")
    off = torch.tensor([0, 20, M], device="cuda")
    o, p, d, e, pl = q(M), q(N), q(M), q(M, mx.elem_code_bytes("e5m2", K)), q(M)
    back = torch.zeros((M, K), device="cuda")
    return {
        "quantize": (lambda: mx.mx_quantize(wide, "floor", *pl[:2]), pl[:2]),
        "quantize_mbs": (lambda: mx.mx_quantize_mbs(x, "oas", *o), o),
        "pair": (lambda: mx.mx_quantize_mbs_pair(x, w, "oas", o, p), o + p),
        "dynamic": (lambda: mx.mx_quantize_mbs_dynamic(x, "oas", 0, 16, 16, *d), d),
        "elem": (lambda: mx.mx_quantize_elem(x, "e5m2", "oas", True, *e), e),
        "elem no words": (lambda: mx.mx_quantize_elem(x, "e5m2", "oas", False, e[0], e[1]), e[:2]),
        "dequantize": (lambda: mx.mx_dequantize(*a, "f32", out=back), (back,)),
        "gemm": (lambda: mx.mx_gemm(a[0], a[1], b[0], b[1], "bf16", out=c), (big,)),
        "gemm_mbs": (lambda: mx.mx_gemm_mbs(*a, b[0], b[1], None, torch.float32, out=f), (f,)),
        "fused": (lambda: mx.mx_gemm_mbs_quantize_a(x, "oas", *b, "bf16", out=c), (big,)),
        "grouped": (lambda: mx.mx_gemm_mbs_grouped(*a, *b, off, N // 2, "f32", out=half), (half,)),
        "gemm_elem": (lambda: mx.mx_gemm_mbs_elem("e2m3", *ea, "e3m2", *eb, "f32", out=f), (f,)),
        "grouped_elem": (lambda: mx.mx_gemm_mbs_elem_grouped("e2m3", *ea, "e3m2", *eb, off, N // 2, "f32", out=half), (half,)),
    }


class Served:
    """A native marshaller that keeps what each of its functions returned."""

    def __init__(self, native):
        self.native, self.returned = native, []

    def __getattr__(self, name):
        def call(*args):
            self.returned.append(getattr(self.native, name)(*args))
            return self.returned[-1]

        return call


def test_same_outputs(mx, monkeypatch):
    made = calls(mx)
    for name, (call, outputs) in made.items():
        got, recorder = [], Served(mx.binding._native)
        for native in (recorder, None):
            for t in outputs:
                t.zero_()
            with monkeypatch.context() as m:
                m.setattr(mx.binding, "_native", native)
                call()
            got.append([t.clone() for t in outputs])
        assert recorder.returned == [0], (name, "declined")
        assert all(torch.equal(s, t) for s, t in zip(*got)) and any(bool(t.any()) for t in got[0]), name


def test_same_errors(mx, monkeypatch):
    x = torch.zeros((4, 512), dtype=torch.bfloat16, device="cuda")
    a, b = mx.mx_quantize_mbs(x), mx.mx_quantize_mbs(torch.zeros((8, 512), dtype=torch.bfloat16, device="cuda"))
    f = torch.zeros((4, 8), device="cuda")
    bad = [lambda: mx.mx_quantize_mbs(x.float(), "oas", *a), lambda: mx.mx_quantize_mbs(x, "oas", a[0], a[1], a[2][:, :1]),
           lambda: mx.mx_quantize_mbs(x, "none", *a), lambda: mx.mx_quantize_mbs(x, 7, *a), lambda: mx.mx_quantize_mbs(x.t(), "oas", *a),
           lambda: mx.mx_gemm_mbs(*a, *b, "f32", out=f.t()), lambda: mx.mx_gemm_mbs(*a, *b, "bf16", out=f), lambda: mx.mx_gemm_mbs(*a, *b, "f16", out=f),
           lambda: mx.mx_gemm_mbs(a[0], None, a[2], *b, "f32", out=f), lambda: mx.mx_gemm_mbs(None, a[1], a[2], *b, "f32", out=f),
           lambda: mx.mx_gemm_mbs(a[0][:, :8], a[1], a[2], *b, "f32", out=f), lambda: mx.mx_gemm_mbs(a[0][:, 1:17], a[1], a[2], b[0][:, :16], b[1], b[2], "f32", out=f),
           lambda: mx.mx_gemm_mbs_grouped(*a, *b, torch.zeros(2, device="cuda"), 8, "f32", out=f),
           lambda: mx.mx_gemm_mbs_elem("e4m3", *a, "e4m3", *b, "f32", out=f)]
    for i, call in enumerate(bad):
        raised = []
        for native in (mx.binding._native, None):
            with monkeypatch.context() as m, pytest.raises(Exception) as e:
                m.setattr(mx.binding, "_native", native)
                call()
            raised.append((type(e.value), str(e.value)))
        assert raised[0] == raised[1], (i, raised)


def test_declines(mx):
    native = mx.binding._native
    x = torch.ones((4, 512), dtype=torch.bfloat16, device="cuda")
    q = (u8(4, 256), u8(4, 16), u8(4, 4))

    class Sub(torch.Tensor):
        pass

    assert native.quantize_mbs(x, "oas", *q) == 0
    for args in ((x.as_subclass(Sub), "oas", *q), (x.cpu(), "oas", *q), (x, 2, *q), (x, "oas", q[0], q[1], None), (x, "oas", *q[:2]),
                 (x.t(), "oas", *q), (x, "oas", q[0][:, ::2], q[1], q[2])):
        assert native.quantize_mbs(*args) is None, args[1:2]
    # inside a transform the tensor is a wrapper without an address: declined, and the Python path raises as it always has
    with pytest.raises(Exception):
        torch.vmap(lambda v: mx.mx_quantize_mbs(v, "oas", *q)[0])(x.unsqueeze(0))


def test_pair_outputs_of_other_lengths(mx):
    """Outputs are given per tensor: an empty tuple asks for them to be allocated, any other number than three is refused."""
    x = torch.randn((4, 512), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda").to(torch.bfloat16)
    q = lambda: (u8(4, 256), u8(4, 16), u8(4, 4))  # noqa: E731
    want = mx.mx_quantize_mbs(x, "oas")
    o0, o1 = mx.mx_quantize_mbs_pair(x, x, "oas", (), q())
    assert all(torch.equal(s, t) for o in (o0, o1) for s, t in zip(o, want, strict=True))
    for out0, out1 in (((), q() + q()), (q()[:2], q()[:1] + q()), (q() + q()[:1], q()[:2])):
        with pytest.raises(TypeError):
            mx.mx_quantize_mbs_pair(x, x, "oas", out0, out1)
