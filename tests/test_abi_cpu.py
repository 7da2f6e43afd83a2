"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol the
header declares, and rejects bad arguments before touching a device."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "mx4.h")
INTERNAL_HEADER = os.path.join(ROOT, "paper_2603_08713_amd", "csrc", "mx_internal.h")


@pytest.fixture(scope="module")
def lib():
    from paper_2603_08713_amd import build as mxbuild
    from paper_2603_08713_amd import binding

    if not os.path.exists(mxbuild.LIB):
        mxbuild.build()
    return binding.load_library()


A16 = 0x10000  # fake, suitably aligned device addresses: rejected calls never dereference them


def declared_functions(header=HEADER):
    text = open(header).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    text = re.sub(r"//[^\n]*", "", text)
    return sorted(set(re.findall(r"\b(mx_[a-z0-9_]+)\s*\(", text)))


def test_header_symbols_are_exported(lib):
    names = declared_functions()
    assert {"mx_quantize", "mx_quantize_oas", "mx_quantize_mbs", "mx_quantize_mbs_dynamic", "mx_quantize_mbs_pair", "mx_gemm_mbs_quantize_a", "mx_dequantize", "mx_gemm", "mx_gemm_mbs",
            "mx_gemm_mbs_grouped", "mx_quantize_elem", "mx_gemm_mbs_elem", "mx_dequantize_elem", "mx_status_string", "mx_version"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n


def test_every_exported_symbol_is_declared(lib):
    """The library exports the public ABI and the development entry points of csrc/mx_internal.h (each a public
    call with one more argument; no switches, no state) and nothing else of its own."""
    import subprocess

    from paper_2603_08713_amd import build as mxbuild

    internal = declared_functions(INTERNAL_HEADER)
    assert internal and all(n.startswith("mx_internal_") for n in internal)
    for n in internal:
        assert hasattr(lib, n), n
    out = subprocess.run(["nm", "-D", "--defined-only", mxbuild.LIB], stdout=subprocess.PIPE, text=True, check=True).stdout
    exported = {l.split()[-1] for l in out.splitlines() if re.search(r" [TW] mx_", l)}
    assert exported == set(declared_functions()) | set(internal), exported ^ (set(declared_functions()) | set(internal))
    assert not any("set_" in n for n in exported)


def test_quantize_rejects_rows_longer_than_its_32_bit_columns(lib):
    K = (1 << 30) + 32
    assert lib.mx_quantize(A16, 1, K, K, 0, A16, A16, None) == -1
    assert lib.mx_quantize_mbs(A16, 1, K, K, 2, A16, A16, A16, None) == -1
    assert lib.mx_quantize_elem(1, A16, 1, K, K, 2, 0, A16, A16, None, None) == -1
    assert lib.mx_internal_quantize(A16, 1, K, K, 0, 0, 0, A16, A16, None, None) == -1


def test_lut_entry_points_reject_bad_arguments(lib):
    assert lib.mx_mbs_lut_build(None, None) == -2
    assert lib.mx_mbs_lut_build(A16 + 2, None) == -3
    q = lib.mx_quantize_mbs_dynamic_lut
    assert q(A16, 4, 48, 48, 2, A16, 1, A16, A16, A16, None) == -1       # K % 32
    assert q(A16, 4, 64, 64, 2, None, 1, A16, A16, A16, None) == -2      # no table
    assert q(A16, 4, 64, 64, 2, A16 + 4, 1, A16, A16, A16, None) == -3   # table misaligned
    assert q(A16, 4, 64, 64, 2, A16, 1, A16, A16, None, None) == -2      # mbs required
    assert q(A16, 0, 64, 64, 2, A16, 1, A16, A16, A16, None) == 0
    s = lib.mx_quantize_mbs_dynamic_lut_static                            # the same checks, before any GPU call
    assert s(A16, 4, 48, 48, 2, 1, A16, A16, A16, None) == -1
    assert s(A16, 4, 64, 64, 2, 1, A16, A16, None, None) == -2
    assert s(A16, 0, 64, 64, 2, 1, A16, A16, A16, None) == 0


def test_gemm_plan_names_the_kernel_a_problem_takes(lib):
    """The planner is host code: which form and tile shape the dispatcher picks, per configuration of the workload
    list, without launching anything."""
    import ctypes

    def plan(M, N, K, a=1, b=1, grouped=0):
        buf = ctypes.create_string_buffer(512)
        assert lib.mx_internal_gemm_plan(M, N, K, a, b, grouped, buf, 512) == 0
        return buf.value.decode()

    big = plan(8192, 28672, 8192)
    assert "fast form" in big and "256x128 tile" in big and "64x64" in big and "A and B" in big
    assert "128x32" in plan(8192, 28672, 8192, 1, 0) and "MBS words on A" in plan(8192, 28672, 8192, 1, 0)
    assert "256x256" in plan(8192, 28672, 8192, 0, 0) and "no MBS" in plan(8192, 28672, 8192, 0, 0)
    assert "128x128" in plan(2048, 2048, 2048)                      # too few large tiles for 256 compute units
    assert "few rows" in plan(16, 4096, 4096)                       # decode
    assert "general form" in plan(32768, 2880, 2880, 1, 1, 1)       # grouped, K % 512 != 0
    assert "tiles of 64 rows and 16 columns, single scale bytes" in plan(512, 512, 2016)           # K % 64 == 32: few-row kernel ...
    assert "row pieces through registers" in plan(4000, 4000, 2016) and "single" not in plan(4000, 4000, 2016)  # ... and general form
    assert "pairs of scale bytes" in plan(16, 4096, 2880) and "scale bytes" not in plan(16, 4096, 4096)
    assert lib.mx_internal_gemm_plan(8, 8, 48, 1, 1, 0, ctypes.create_string_buffer(8), 8) == -1   # K % 32
    assert lib.mx_internal_gemm_plan(8, 8, 64, 1, 1, 0, None, 0) == -1
    # grouped: the choice goes by the rows per group
    assert "few rows per group" in plan(32 * 32, 2880, 2880, grouped=32)
    assert "general form" in plan(32 * 32 + 1, 2880, 2880, grouped=32)
    # ... and by what fits a launch of fewer than 2^32 work-items
    assert "few rows per group" in plan(2048, 1 << 22, 64, grouped=64) and "general form" in plan(2048, 1 << 23, 64, grouped=64)
    assert "few rows per group" in plan(64, 1 << 21, 32, grouped=64) and "general form" in plan(64, 1 << 23, 32, grouped=64)
    import paper_2603_08713_amd as mx

    assert "few rows per group" in mx.gemm_plan(256, 2880, 2880, grouped=True, num_groups=32)
    # few rows, K % 512 != 0: the few-row kernel as far as its rounds of narrow workgroups are cheaper than the main kernel's tiles
    for M, N, K, few in ((64, 8192, 1088, 1), (64, 28672, 1088, 0), (1, 14336, 2880, 1), (64, 14336, 2880, 1), (32, 28672, 2880, 0),
                         (64, 4096, 4128, 1), (64, 28672, 4128, 0), (16, 28672, 4128, 1), (64, 28672, 4096, 1), (1, 1 << 30, 32, 0)):
        assert ("few rows" in plan(M, N, K)) == bool(few), (M, N, K)
    assert "few rows" in mx.gemm_plan(16, 4096, 4096) and "few rows" not in mx.gemm_plan(65, 4096, 4096)


def test_binding_output_type_names():
    """Whatever equals a type code, a name or a torch dtype names the output type, hashable or not."""
    import numpy as np
    import torch

    import paper_2603_08713_amd as mx
    from paper_2603_08713_amd import binding

    for code, dtype, names in ((mx.MX_OUT_F32, torch.float32, ("f32", "fp32", torch.float32)), (mx.MX_OUT_BF16, torch.bfloat16, ("bf16", torch.bfloat16))):
        for name in names + (code, float(code), np.int64(code), np.array(code), torch.tensor(code)):
            assert binding._out_dtype(name) == (code, dtype), name
    for name in ("f16", 7, None, torch.float16, [], np.array(9)):
        with pytest.raises(ValueError):
            binding._out_dtype(name)


def test_binding_leaves_missing_scales_to_the_library(monkeypatch):
    """An operand without its scale array: the library's own status, and nothing at all for an empty product."""
    import torch

    import paper_2603_08713_amd as mx
    from paper_2603_08713_amd import binding

    monkeypatch.setattr(binding, "_stream", lambda: 0)
    codes, scales = torch.zeros((4, 32), dtype=torch.uint8), torch.zeros((4, 2), dtype=torch.uint8)
    for a_scales, b_scales in ((None, scales), (scales, None)):
        for call in (lambda a: mx.mx_gemm(a, a_scales, codes, b_scales), lambda a: mx.mx_gemm_mbs(a, a_scales, None, codes, b_scales, None)):
            with pytest.raises(mx.MxError):
                call(codes)
            assert call(codes[:0]).shape == (0, 4)
    with pytest.raises(mx.MxError):
        mx.mx_dequantize(codes, None)
    assert mx.mx_dequantize(codes[:0], None).shape == (0, 64)


def test_version_and_status_strings(lib):
    assert lib.mx_version() >= 100
    seen = set()
    for code in (0, -1, -2, -3, -4, -5):
        s = lib.mx_status_string(code).decode()
        assert s and s not in seen
        seen.add(s)
    assert "unknown" in lib.mx_status_string(-99).decode()


def test_quantize_argument_errors(lib):
    q = lib.mx_quantize
    assert q(A16, 4, 48, 48, 0, A16, A16, None) == -1          # K % 32
    assert q(A16, -1, 64, 64, 0, A16, A16, None) == -1         # negative rows
    assert q(A16, 4, 64, 32, 0, A16, A16, None) == -1          # ldx < K
    assert q(A16, 4, 64, 64, 7, A16, A16, None) == -1          # bad rule
    assert q(None, 4, 64, 64, 0, A16, A16, None) == -2
    assert q(A16, 4, 64, 64, 0, None, A16, None) == -2
    assert q(A16, 4, 64, 64, 0, A16, None, None) == -2
    assert q(A16 + 2, 4, 64, 64, 0, A16, A16, None) == -3      # x misaligned
    assert q(A16, 4, 64, 68, 0, A16, A16, None) == -3          # ldx % 8
    assert q(A16, 4, 64, 64, 0, A16 + 4, A16, None) == -3      # codes misaligned
    assert q(A16, 0, 64, 64, 0, A16, A16, None) == 0           # empty is a no-op
    assert lib.mx_quantize_oas(A16, 4, 40, 40, A16, A16, None) == -1
    assert lib.mx_quantize_mbs(A16, 4, 64, 64, 2, A16, A16, None, None) == -2   # mbs required
    assert lib.mx_quantize_mbs(A16, 0, 64, 64, 2, A16, A16, None, None) == 0
    p = lib.mx_quantize_mbs_pair
    assert p(A16, 4, 64, A16, A16, A16, A16, 4, 64, A16, A16, A16, 48, 2, None) == -1      # K % 32
    assert p(A16, 4, 64, A16, A16, A16, A16, 4, 32, A16, A16, A16, 64, 2, None) == -1      # second ld < K
    assert p(A16, 4, 64, A16, A16, None, A16, 4, 64, A16, A16, A16, 64, 2, None) == -2
    assert p(A16, 4, 64, A16, A16, A16, A16 + 2, 4, 64, A16, A16, A16, 64, 2, None) == -3
    assert p(A16, 0, 64, A16, A16, A16, A16, 0, 64, A16, A16, A16, 64, 2, None) == 0
    d = lib.mx_quantize_mbs_dynamic
    assert d(A16, 4, 64, 64, 2, 0, 257, 16, A16, A16, A16, None) == -1          # too many candidates
    assert d(A16, 4, 64, 64, 2, 0, -1, 16, A16, A16, A16, None) == -1
    assert d(A16, 4, 64, 64, 2, 1 << 20, 16, 16, A16, A16, A16, None) == -1     # offsets out of range
    assert d(A16, 4, 64, 64, 2, 0, 16, -(1 << 20), A16, A16, A16, None) == -1
    assert d(A16, 4, 48, 48, 2, 0, 16, 16, A16, A16, A16, None) == -1           # K % 32
    assert d(A16, 4, 64, 64, 2, 0, 16, 16, A16, A16, None, None) == -2          # mbs required
    assert d(A16, 0, 64, 64, 2, 0, 16, 16, A16, A16, A16, None) == 0


def test_gemm_quantize_a_argument_errors(lib):
    f = lib.mx_gemm_mbs_quantize_a
    ok = (A16, 512, 2, 1, A16, A16, A16, 16, 64, 512, 0, A16, 64, None)

    def call(**kw):
        names = ("a", "lda", "rule", "a_mbs", "bc", "bs", "bm", "M", "N", "K", "dt", "C", "ldc", "stream")
        args = dict(zip(names, ok))
        args.update(kw)
        return f(*[args[n] for n in names])

    assert call(K=48, lda=48) == -1
    assert call(lda=256) == -1              # lda < K
    assert call(ldc=32) == -1               # ldc < N
    assert call(rule=9) == -1
    assert call(dt=3) == -1
    assert call(M=0) == 0 and call(N=0) == 0
    assert call(a=None) == -2 and call(bc=None) == -2 and call(bs=None) == -2 and call(C=None) == -2
    assert call(a=A16 + 2) == -3 and call(lda=516) == -3 and call(bc=A16 + 8) == -3
    assert call(M=65) == -4                 # shapes the few-row kernel does not cover
    assert call(K=544, lda=544) == -4
    assert call(K=16384, lda=16384) == -4
    assert call(bs=A16 + 4) == -4
    assert call(bm=A16 + 2) == -4


def test_dequantize_argument_errors(lib):
    d = lib.mx_dequantize
    assert d(A16, A16, None, 4, 48, 0, A16, 48, None) == -1
    assert d(A16, A16, None, 4, 64, 5, A16, 64, None) == -1
    assert d(A16, A16, None, 4, 64, 0, A16, 32, None) == -1
    assert d(None, A16, None, 4, 64, 0, A16, 64, None) == -2
    assert d(A16, A16, None, 4, 64, 0, None, 64, None) == -2
    assert d(A16, A16, None, 4, 64, 0, A16 + 2, 64, None) == -3
    assert d(A16, A16, None, 0, 64, 0, A16, 64, None) == 0


def test_gemm_argument_errors(lib):
    g = lib.mx_gemm
    assert g(A16, A16, A16, A16, 8, 8, 48, 0, A16, 8, None) == -1
    assert g(A16, A16, A16, A16, -8, 8, 64, 0, A16, 8, None) == -1
    assert g(A16, A16, A16, A16, 8, 8, 64, 0, A16, 4, None) == -1     # ldc < N
    assert g(A16, A16, A16, A16, 8, 8, 64, 9, A16, 8, None) == -1
    assert g(None, A16, A16, A16, 8, 8, 64, 0, A16, 8, None) == -2
    assert g(A16, A16, A16, A16, 8, 8, 64, 0, None, 8, None) == -2
    assert g(A16 + 8, A16, A16, A16, 8, 8, 64, 0, A16, 8, None) == -3
    assert g(A16, A16, A16, A16, 0, 8, 64, 0, A16, 8, None) == 0
    m = lib.mx_gemm_mbs
    assert m(A16, A16, None, A16, A16, None, 8, 8, 40, 0, A16, 8, None) == -1
    assert m(A16, A16, None, A16, A16, None, 8, 0, 64, 0, A16, 8, None) == 0
    gg = lib.mx_gemm_mbs_grouped
    assert gg(A16, A16, None, A16, A16, None, 2, None, 8, 8, 64, 0, A16, 8, None) == -2
    assert gg(A16, A16, None, A16, A16, None, -1, A16, 8, 8, 64, 0, A16, 8, None) == -1
    assert gg(A16, A16, None, A16, A16, None, 0, A16, 8, 8, 64, 0, A16, 8, None) == 0


def test_elem_argument_errors(lib):
    q = lib.mx_quantize_elem
    E4, E5, E23, E2M1 = 1, 2, 3, 0
    assert q(E4, A16, 4, 48, 48, 2, 1, A16, A16, A16, None) == -1      # K % 32
    assert q(E2M1, A16, 4, 64, 64, 2, 1, A16, A16, A16, None) == -1    # the 4-bit format has its own entry points
    assert q(9, A16, 4, 64, 64, 2, 1, A16, A16, A16, None) == -1       # bad element format
    assert q(E4, A16, 4, 64, 64, 5, 1, A16, A16, A16, None) == -1      # bad rule
    assert q(E4, A16, 4, 64, 64, 2, 1, A16, A16, None, None) == -2     # MBS words wanted, no array
    assert q(E4, None, 4, 64, 64, 2, 0, A16, A16, None, None) == -2
    assert q(E5, A16, 4, 64, 64, 2, 0, A16 + 4, A16, None, None) == -3  # codes 8-byte aligned
    assert q(E23, A16, 0, 64, 64, 2, 0, A16, A16, None, None) == 0     # the 6-bit formats quantize too
    assert q(E4, A16, 0, 64, 64, 2, 0, A16, A16, None, None) == 0
    qd = lib.mx_quantize_elem_mbs_dynamic
    assert qd(E4, A16, 4, 48, 48, 2, 0, 16, 16, A16, A16, A16, None) == -1     # K % 32
    assert qd(E2M1, A16, 4, 64, 64, 2, 0, 16, 16, A16, A16, A16, None) == -1   # the 4-bit format has its own entry point
    assert qd(E4, A16, 4, 64, 64, 2, 0, 257, 16, A16, A16, A16, None) == -1    # too many candidates
    assert qd(E4, A16, 4, 64, 64, 2, 0, 16, 70000, A16, A16, A16, None) == -1  # stride out of range
    assert qd(E4, A16, 4, 64, 64, 2, 0, 16, 16, A16, A16, None, None) == -2    # the words have nowhere to go
    assert qd(E5, A16, 4, 64, 64, 2, 0, 16, 16, A16 + 4, A16, A16, None) == -3
    assert qd(E23, A16, 0, 64, 64, 2, 0, 16, 16, A16, A16, A16, None) == 0
    d = lib.mx_dequantize_elem
    assert d(E4, A16, A16, None, 4, 48, 0, A16, 48, None) == -1     # K % 32
    assert d(E2M1, A16, A16, None, 4, 64, 0, A16, 64, None) == -1   # the 4-bit format has its own entry point
    assert d(E4, A16, A16, None, 4, 64, 0, A16, 32, None) == -1     # ldo < K
    assert d(E4, A16, A16, None, 4, 64, 5, A16, 64, None) == -1     # bad output type
    assert d(E4, None, A16, None, 4, 64, 0, A16, 64, None) == -2
    assert d(E5, A16 + 4, A16, None, 4, 64, 0, A16, 64, None) == -3
    assert d(E23, A16, A16, None, 4, 48, 0, A16, 48, None) == -1    # the 6-bit formats: the same checks
    assert d(E23, A16, A16, None, 0, 64, 0, A16, 64, None) == 0
    assert d(E4, A16, A16, None, 0, 64, 0, A16, 64, None) == 0
    g = lib.mx_gemm_mbs_elem
    assert g(E4, A16, A16, None, E4, A16, A16, None, 8, 8, 48, 0, A16, 8, None) == -1
    assert g(E2M1, A16, A16, None, E4, A16, A16, None, 8, 8, 128, 0, A16, 8, None) == -1
    assert g(E4, A16, A16, None, E5, A16, A16, None, 8, 8, 128, 0, A16, 4, None) == -1   # ldc < N
    assert g(E4, None, A16, None, E5, A16, A16, None, 8, 8, 128, 0, A16, 8, None) == -2
    assert g(E4, A16, A16, None, E5, A16, A16, None, 8, 8, 128, 0, None, 8, None) == -2
    assert g(E4, A16, A16, None, E5, A16, A16, None, 8, 8, 64, 0, A16, 8, None) == -4    # K % 128
    assert g(E4, A16, A16, None, E5, A16, A16 + 2, None, 8, 8, 128, 0, A16, 8, None) == -4  # scale rows not dword-aligned
    assert g(E4, A16, A16, None, E23, A16, A16, None, 8, 8, 128, 0, A16, 8, None) == -4  # 6-bit formats
    assert g(E4, A16, A16, None, E5, A16, A16, None, 0, 8, 128, 0, A16, 8, None) == 0
    gg = lib.mx_gemm_mbs_elem_grouped
    assert gg(E4, A16, A16, None, E5, A16, A16, None, -1, A16, 8, 8, 128, 0, A16, 8, None) == -1   # negative group count
    assert gg(E4, A16, A16, None, E5, A16, A16, None, 2, None, 8, 8, 128, 0, A16, 8, None) == -2   # no offsets
    assert gg(E4, A16, A16, None, E5, A16, A16, None, 2, A16, 8, 8, 48, 0, A16, 8, None) == -1     # K % 32
    assert gg(E4, A16, A16, None, E5, A16, A16, None, 2, A16, 8, 8, 64, 0, A16, 8, None) == -4     # K % 128
    assert gg(E4, A16, A16, None, E23, A16, A16, None, 2, A16, 8, 8, 128, 0, A16, 8, None) == -4   # 8-bit with 6-bit
    assert gg(E23, A16, A16, None, E23, A16, A16, None, 0, None, 8, 8, 128, 0, A16, 8, None) == 0  # no groups: nothing to do
    assert gg(E4, A16, A16, None, E5, A16, A16, None, 2, A16, 0, 8, 128, 0, A16, 8, None) == 0


def test_fp8_dequantizer_shortcut_is_exact():
    """The MXFP8 / MXFP6 dequantizer's result is defined through fp64 (quotient rounded at 53 bits, then to fp32).
    Where every intermediate is a normal fp32 number the kernel divides once per run, r = RN(1 / F), and per element
    computes q = RN(t r), rem = t - q F (exact, one fma), q' = RN(q + rem r).  With exact rationals: q' is the
    correctly rounded t / F, and equals the fp64 route, for every pair of code value (FP8 and FP6 formats) and MBS
    word; a power-of-two block scale commutes with all of it, so one binade per mantissa covers every scale byte
    of the shortcut's range."""
    import math
    from fractions import Fraction

    import numpy as np

    def rn32(x):  # Fraction -> nearest fp32 (ties to even), normal range, as a Fraction
        if x == 0:
            return Fraction(0)
        e = math.floor(math.log2(x))
        while Fraction(2) ** e > x:
            e -= 1
        while Fraction(2) ** (e + 1) <= x:
            e += 1
        n = x / Fraction(2) ** (e - 23)
        fl = n.numerator // n.denominator
        rem = n - fl
        if rem > Fraction(1, 2) or (rem == Fraction(1, 2) and fl % 2 == 1):
            fl += 1
        return fl * Fraction(2) ** (e - 23)

    def values(mbits, bias, top):
        out = set()
        for c in range(1, top + 1):
            e, m = c >> mbits, c & ((1 << mbits) - 1)
            out.add(Fraction(m, 1 << mbits) * Fraction(2) ** (1 - bias) if e == 0 else (1 + Fraction(m, 1 << mbits)) * Fraction(2) ** (e - bias))
        return out

    vals = set()
    for fmt in ((3, 7, 0x7E), (2, 15, 0x7B), (3, 1, 0x1F), (2, 3, 0x1F)):  # E4M3, E5M2, E2M3, E3M2
        vals |= values(*fmt)
    mantissas = sorted({v / Fraction(2) ** math.floor(math.log2(v)) for v in vals})
    assert mantissas == [Fraction(8 + k, 8) for k in range(8)]
    for t in mantissas:
        for m8 in range(256):
            F = 1 + Fraction(m8, 256)
            r = rn32(1 / F)
            q0 = rn32(t * r)
            rem = t - q0 * F
            assert rem == 0 or rn32(abs(rem)) == abs(rem)      # the fma returns it exactly
            q1 = q0 + rem * r
            q1 = rn32(q1) if q1 > 0 else Fraction(0)
            assert q1 == rn32(t / F), (t, m8)
    # and the correctly rounded quotient is what the fp64 route gives
    v = np.array([float(x) for x in sorted(vals)], np.float64)[:, None]
    F = 1.0 + np.arange(256, dtype=np.float64)[None, :] / 256.0
    via64 = (v / F).astype(np.float32)
    direct = v.astype(np.float32) / F.astype(np.float32)  # IEEE fp32 division: correctly rounded
    assert direct.dtype == np.float32 and np.array_equal(via64, direct)


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    from paper_2603_08713_amd import binding

    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_LIB_PATH", str(tmp_path / "nope.so"))
    with pytest.raises(ImportError):
        binding.load_library()


def test_product_path_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_2603_08713_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                text = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in text.replace("test oracle", ""), f
