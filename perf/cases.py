"""The work that a user of this library has it do, as cases that can be timed and compared.

The ranges follow the workloads of the benchmark and of the tests: Llama-3-8B and Llama-3-70B FFN layers (whole
steps that quantize both operands, and inference with weights quantized beforehand), decode with 1 to 64 rows, the
mixture-of-experts layer with K = 2880 that ends in half a macro block, the 8-bit and 6-bit element formats, and the
offline side: weights quantized with searched words and dequantized again.  Weights are the stored operand of a layer
and therefore prepared; activations arrive as bf16 in every pass.

kinds (each a range that `draw` samples):
  step      quantize A and W in one launch, then the MBS GEMM: a training-like pass, or a layer whose weights change
  linear    quantize A, then the GEMM with a prepared weight, with or without MBS words: prefill of a prompt
  decode    the few-row GEMM with the activations quantized inside it
  moe       quantize the routed rows, then the grouped GEMM over the experts, for prefill and for decode batches
  elem      quantize A into an 8-bit or 6-bit format, then the GEMM of that format with a prepared weight
  weights   quantize a weight offline with searched MBS words, and dequantize it (what an error report does)
"""
from __future__ import annotations

import math

import torch

import paper_2603_08713_amd as mx
from paper_2603_08713_amd import synth

BF16_BYTES = 2.0


def listed():
    return [
        # the configuration of the smoke test: two launches of a few microseconds, fp32 output
        dict(name="step_tiny", kind="step", M=64, N=256, K=512, out="f32"),
        # one decode step of 16 sequences, attention projection of the 8B model
        dict(name="decode_16x4096", kind="decode", M=16, N=4096, K=4096, out="bf16"),
        # the same batch against the FFN up-projection
        dict(name="decode_16x14336", kind="decode", M=16, N=14336, K=4096, out="bf16"),
        # prefill of one prompt of odd length, attention projection
        dict(name="linear_prompt_333", kind="linear", M=333, N=4096, K=4096, mbs=True, out="bf16"),
        # prefill of a large batch, FFN up-projection of the 8B model, weights quantized offline
        dict(name="linear_8b", kind="linear", M=4096, N=14336, K=4096, mbs=True, out="bf16"),
        # the benchmark's headline step, FFN of the 70B model
        dict(name="step_70b", kind="step", M=8192, N=28672, K=8192, out="bf16"),
        # plain MXFP4 (no MBS words) on a ragged shape: K ends in half a macro block, N and M are odd
        dict(name="linear_plain_ragged", kind="linear", M=1777, N=5001, K=2880, mbs=False, out="f32"),
        # mixture-of-experts layer, a prefill batch of 8192 tokens routed to 4 of 32 experts
        dict(name="moe_prefill", kind="moe", tokens=8192, experts=32, top_k=4, dim=2880, elem="e2m1", out="bf16"),
        # the same layer when 64 sequences decode: a few rows for every expert
        dict(name="moe_decode", kind="moe", tokens=64, experts=32, top_k=4, dim=2880, elem="e2m1", out="bf16"),
        # MXFP8 and MXFP6 layers
        dict(name="elem_e4m3_8b", kind="elem", elem="e4m3", M=4096, N=14336, K=4096, mbs=True, out="bf16"),
        dict(name="elem_e2m3_prompt", kind="elem", elem="e2m3", M=1024, N=4096, K=4096, mbs=True, out="bf16"),
        # offline: the 8B FFN weight with searched words, and back to bf16
        dict(name="weights_8b", kind="weights", M=14336, K=4096, out="bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(x, m, lo):
    return max(lo, x // m * m)


def draw(rng):
    kind = rng.choice(["step", "linear", "linear", "decode", "decode", "moe", "moe", "elem", "elem", "weights"])
    out = rng.choice(["bf16", "bf16", "bf16", "f32"])
    if kind == "step":
        return dict(kind=kind, M=_log(rng, 64, 8192), N=_log(rng, 256, 14336), K=_mult(_log(rng, 512, 8192), 32, 512), out=out)
    if kind == "linear":
        # model dimensions are multiples of 512 more often than not
        step = rng.choice([512, 512, 64, 32])
        return dict(kind=kind, M=_log(rng, 65, 4096), N=_log(rng, 1024, 16384), K=_mult(_log(rng, 512, 8192), step, 512),
                    mbs=rng.random() < 0.7, out=out)
    if kind == "decode":
        return dict(kind=kind, M=_log(rng, 1, 64), N=_log(rng, 512, 28672), K=_mult(_log(rng, 512, 8192), 512, 512), out=out)
    if kind == "moe":
        elem = rng.choice(["e2m1", "e2m1", "e4m3", "e2m3"])
        return dict(kind=kind, tokens=_log(rng, 8, 8192), experts=rng.choice([8, 16, 32, 64]), top_k=rng.choice([2, 4]),
                    dim=_mult(_log(rng, 768, 3072), 64, 768), elem=elem, out=out)
    if kind == "elem":
        return dict(kind=kind, elem=rng.choice(["e4m3", "e5m2", "e2m3", "e3m2"]), M=_log(rng, 1, 4096), N=_log(rng, 1024, 14336),
                    K=_mult(_log(rng, 512, 8192), rng.choice([512, 512, 128, 64]), 512), mbs=rng.random() < 0.7, out=out)
    return dict(kind="weights", M=_log(rng, 256, 28672), K=_mult(_log(rng, 512, 8192), 32, 512), out=out)


# ---- inputs -----------------------------------------------------------------------------------------------
def _weights(gen, rows, K):
    """N(0, 0.02^2) as the synthetic weights of the benchmark."""
    x = torch.empty((rows, K), dtype=torch.bfloat16, device="cuda")
    step = max(1, (1 << 26) // K)
    for r in range(0, rows, step):
        n = min(step, rows - r)
        x[r:r + n] = torch.randn((n, K), generator=gen, device="cuda") * 0.02
    return x


def _activations(gen, rows, K):
    """Student-t(4) with 1 % of the channels times 20, as the synthetic activations of the benchmark."""
    scale = torch.ones(K, device="cuda")
    scale[torch.randperm(K, generator=gen, device="cuda")[:math.ceil(0.01 * K)]] = 20.0
    x = torch.empty((rows, K), dtype=torch.bfloat16, device="cuda")
    step = max(1, (1 << 25) // K)
    for r in range(0, rows, step):
        n = min(step, rows - r)
        z = torch.randn((n, K), generator=gen, device="cuda")
        u = torch.rand((n, K), generator=gen, device="cuda").clamp_min_(1e-30)
        v = torch.rand((n, K), generator=gen, device="cuda").clamp_min_(1e-30)
        chi2 = -2.0 * (u.log_() + v.log_())  # chi-squared with 4 degrees of freedom
        x[r:r + n] = z * (chi2 / 4.0).clamp_min_(1e-6).rsqrt_() * scale
    return x


def _empty(rows, cols, dtype=torch.uint8):
    return torch.empty((rows, cols), dtype=dtype, device="cuda")


def _quantized_buffers(rows, K, mbs=True, elem="e2m1"):
    code_bytes = K // 2 if elem == "e2m1" else mx.elem_code_bytes(elem, K)
    return (_empty(rows, code_bytes), _empty(rows, K // 32)) + ((_empty(rows, (K + 127) // 128),) if mbs else (None,))


def _c_buffer(case, rows, N):
    return _empty(rows, N, torch.float32 if case["out"] == "f32" else torch.bfloat16)


def prepare(case, seed):
    """Inputs of one pass, the stored weights of the layer and the buffers a serving program keeps."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind, out = case["kind"], case["out"]
    s = dict(kind=kind, out=out)
    if kind == "step":
        M, N, K = case["M"], case["N"], case["K"]
        s.update(a=_activations(gen, M, K), w=_weights(gen, N, K), qa=_quantized_buffers(M, K), qw=_quantized_buffers(N, K),
                 c=_c_buffer(case, M, N))
    elif kind == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        w = _weights(gen, N, K)
        s.update(a=_activations(gen, M, K), mbs=case["mbs"], qa=_quantized_buffers(M, K, case["mbs"]), c=_c_buffer(case, M, N),
                 qw=mx.mx_quantize_mbs(w, "oas") if case["mbs"] else mx.mx_quantize(w, "oas"))
    elif kind == "decode":
        M, N, K = case["M"], case["N"], case["K"]
        s.update(a=_activations(gen, M, K), qw=mx.mx_quantize_mbs(_weights(gen, N, K), "oas"), c=_c_buffer(case, M, N))
    elif kind == "moe":
        experts, dim, elem = case["experts"], case["dim"], case["elem"]
        offsets, _ = synth.zipf_topk_routing(case["tokens"], experts, case["top_k"], 1.1, seed)
        rows = case["tokens"] * case["top_k"]
        w = _weights(gen, experts * dim, dim)
        s.update(a=_activations(gen, rows, dim), elem=elem, N=dim, c=_c_buffer(case, rows, dim),
                 offsets=torch.from_numpy(offsets).cuda(), qa=_quantized_buffers(rows, dim, True, elem),
                 qw=mx.mx_quantize_mbs(w, "oas") if elem == "e2m1" else mx.mx_quantize_elem(w, elem, "oas", True))
    elif kind == "elem":
        M, N, K, elem = case["M"], case["N"], case["K"], case["elem"]
        s.update(a=_activations(gen, M, K), elem=elem, mbs=case["mbs"], qa=_quantized_buffers(M, K, case["mbs"], elem),
                 qw=mx.mx_quantize_elem(_weights(gen, N, K), elem, "oas", case["mbs"]), c=_c_buffer(case, M, N))
    else:
        M, K = case["M"], case["K"]
        s.update(w=_weights(gen, M, K), qw=_quantized_buffers(M, K), back=_c_buffer(case, M, K))
    return s


def run(s):
    """One pass through the library's entry points; everything is enqueued on the current stream."""
    kind, out = s["kind"], s["out"]
    if kind == "step":
        qa, qw = s["qa"], s["qw"]
        mx.mx_quantize_mbs_pair(s["a"], s["w"], "oas", qa, qw)
        mx.mx_gemm_mbs(*qa, *qw, out, out=s["c"])
        return dict(a_codes=qa[0], a_scales=qa[1], a_mbs=qa[2], w_codes=qw[0], w_scales=qw[1], w_mbs=qw[2], c=s["c"])
    if kind == "linear":
        qa, qw = s["qa"], s["qw"]
        if s["mbs"]:
            mx.mx_quantize_mbs(s["a"], "oas", *qa)
            mx.mx_gemm_mbs(*qa, *qw, out, out=s["c"])
            return dict(a_codes=qa[0], a_scales=qa[1], a_mbs=qa[2], c=s["c"])
        mx.mx_quantize(s["a"], "oas", qa[0], qa[1])
        mx.mx_gemm(qa[0], qa[1], qw[0], qw[1], out, out=s["c"])
        return dict(a_codes=qa[0], a_scales=qa[1], c=s["c"])
    if kind == "decode":
        return dict(c=mx.mx_gemm_mbs_quantize_a(s["a"], "oas", *s["qw"], out, out=s["c"]))
    if kind == "moe":
        qa, qw = s["qa"], s["qw"]
        if s["elem"] == "e2m1":
            mx.mx_quantize_mbs(s["a"], "oas", *qa)
            mx.mx_gemm_mbs_grouped(*qa, *qw, s["offsets"], s["N"], out, out=s["c"])
        else:
            mx.mx_quantize_elem(s["a"], s["elem"], "oas", True, *qa)
            mx.mx_gemm_mbs_elem_grouped(s["elem"], *qa, s["elem"], *qw, s["offsets"], s["N"], out, out=s["c"])
        return dict(a_codes=qa[0], a_scales=qa[1], a_mbs=qa[2], c=s["c"])
    if kind == "elem":
        qa, qw = s["qa"], s["qw"]
        mx.mx_quantize_elem(s["a"], s["elem"], "oas", s["mbs"], *qa)
        mx.mx_gemm_mbs_elem(s["elem"], *qa, s["elem"], *qw, out, out=s["c"])
        return dict(zip(("a_codes", "a_scales", "a_mbs"), qa), c=s["c"]) if s["mbs"] else dict(a_codes=qa[0], a_scales=qa[1], c=s["c"])
    qw = mx.mx_quantize_mbs_dynamic(s["w"], "oas", 0, 16, 16, *s["qw"])
    return dict(codes=qw[0], scales=qw[1], mbs=qw[2], back=mx.mx_dequantize(*qw, out, out=s["back"]))


# ---- what a pass cannot do without ---------------------------------------------------------------------------
def _quantized_bytes(rows, K, mbs=True, elem="e2m1"):
    code = {"e2m1": 0.5, "e2m3": 0.75, "e3m2": 0.75}.get(elem, 1.0)
    return rows * (K * code + K // 32 + ((K + 127) // 128 if mbs else 0))


def work(case):
    kind, esz = case["kind"], 4.0 if case["out"] == "f32" else 2.0
    if kind == "weights":
        M, K = case["M"], case["K"]
        # (a few operations per element; the search's price depends on how it is done)
        return {"bytes": M * K * (BF16_BYTES + esz) + _quantized_bytes(M, K), "flops": 0.0}
    if kind == "moe":
        rows, dim, elem = case["tokens"] * case["top_k"], case["dim"], case["elem"]
        # the weights of every expert that has rows; with few tokens an expert may have none
        busy = min(case["experts"], rows)
        return {"bytes": rows * dim * (BF16_BYTES + esz) + _quantized_bytes(rows, dim, True, elem)
                + busy * _quantized_bytes(dim, dim, True, elem), "flops": 2.0 * rows * dim * dim}
    M, N, K = case["M"], case["N"], case["K"]
    mbs, elem = case.get("mbs", True), case.get("elem", "e2m1")
    total = M * K * BF16_BYTES + M * N * esz + _quantized_bytes(N, K, mbs, elem)
    if kind == "step":
        total += N * K * BF16_BYTES
    if kind != "decode":
        total += _quantized_bytes(M, K, mbs, elem)
    return {"bytes": total, "flops": 2.0 * M * N * K}


def tolerance(case):
    """Codes, scales and words are bytes and stay the same.  C was measured against the same operands multiplied in 64
    bits (and rounded to bf16 where the output is): relative error 1e-7 for fp32 output and 2.5e-5 for bf16, where a last
    bit differs where the fp32 sum lies near a tie; for the 8-bit formats and E3M2, whose products the matrix
    instruction cuts 13 bits below the largest of 16, 1e-4 and 3.6e-4.  Stated: four times that, ten for the sums in
    fp32, whose error grows with K.  Largest difference: 1.6e-6 of the RMS for fp32; for bf16 one last bit, which is up to
    2^-7 of the value (two where the products are cut)."""
    if case["kind"] == "weights":
        # a window whose two best words tie to within the rounding of an fp32 sum may take either: about one window
        # in 10^5, each changing its 128 values by a tenth and a value by at most a step of its grid
        return {"rel": 1e-3, "max": 1.0, "differ": 5e-5}
    cut = case.get("elem") in ("e4m3", "e5m2", "e3m2")
    if case["out"] == "f32":
        return {"rel": 4e-4, "max": 4e-3} if cut else {"rel": 1e-6, "max": 1e-5}
    return {"rel": 1.5e-3, "max": 0.016} if cut else {"rel": 1e-4, "max": 0.008}
