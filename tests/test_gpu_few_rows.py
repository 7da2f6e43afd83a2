"""The few-row GEMM kernel at the edges of its tiles, chunks and forms, against the CPU oracle: shares of K that are
whole chunks of four macro blocks, parts of one and none at all; the four ways E8M0 bytes and MBS words travel (by K and by
the alignment of the arrays); grouped problems with empty groups, groups of one row and of several tile-rows, and with
nearly all rows in one group; the form with the activations quantized inside, bit for bit the quantizer and the GEMM."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_08713_amd as mx_

    mx_.load_library()
    return mx_


def random_operand(rng, rows, K):
    return (rng.integers(0, 256, (rows, K // 2), dtype=np.uint8), rng.integers(110, 140, (rows, K // 32), dtype=np.uint8),
            rng.integers(0, 256, (rows, (K + 127) // 128), dtype=np.uint8))


def dev(a, shift=0):
    """On the GPU, `shift` bytes into an allocation (rows stay contiguous)."""
    flat = torch.zeros(a.size + shift, dtype=torch.uint8, device="cuda")
    flat[shift:] = torch.from_numpy(a.reshape(-1)).cuda()
    return flat[shift:].view(a.shape)


def close(got, want, what):
    # 1e-3 of the RMS is the interface's bound on the fp32 output
    err, rms = np.abs(got.cpu().numpy().astype(np.float64) - want).max(), np.sqrt(np.mean(want ** 2))
    assert err <= 1e-3 * rms, (what, err, rms)


# K: one macro block for some wavefronts and none for others (512), unequal parts of a chunk (1536, 2560), one whole chunk
# each (4096), chunk and a part (6656), two chunks (8192); 2880 and 2016 end inside a macro block; 32 is a single block
@pytest.mark.parametrize("M,N,K", [(1, 17, 512), (16, 4113, 1536), (17, 250, 2560), (33, 8209, 4096), (64, 100, 6656), (5, 40, 8192),
                                   (16, 33, 2880), (50, 4100, 2880), (31, 70, 2016), (3, 16, 32), (64, 257, 64), (9, 31, 192)])
@pytest.mark.parametrize("shift", [0, 2, 1])
def test_few_rows_every_form(mx, oracle, M, N, K, shift):
    """shift: scale and word arrays that start 0, 2 or 1 bytes past a 16-byte boundary."""
    rng = np.random.default_rng(M * 7 + K + shift)
    a, b = random_operand(rng, M, K), random_operand(rng, N, K)
    da, db = [dev(a[0])] + [dev(t, shift) for t in a[1:]], [dev(b[0])] + [dev(t, shift) for t in b[1:]]
    for am, bm in ((True, True), (False, False), (False, True)):
        want = oracle.gemm((a[0], a[1], a[2] if am else None), (b[0], b[1], b[2] if bm else None))
        big = torch.full((M + 2, N + 3), -3.0, dtype=torch.float32, device="cuda")
        out = big[1:M + 1, 1:N + 1]
        mx.mx_gemm_mbs(da[0], da[1], da[2] if am else None, db[0], db[1], db[2] if bm else None, "f32", out=out)
        close(out, want, (M, N, K, shift, am, bm))
        c16 = mx.mx_gemm_mbs(da[0], da[1], da[2] if am else None, db[0], db[1], db[2] if bm else None, "bf16")
        assert torch.equal(c16, out.to(torch.bfloat16))
        big[1:M + 1, 1:N + 1] = -3.0
        assert bool((big == -3.0).all())


@pytest.mark.parametrize("M,N,K,shift", [(33, 8209, 4096, 1), (64, 8300, 1088, 0), (17, 8193, 64, 2), (64, 12301, 1056, 0)])
def test_few_rows_in_more_than_one_round(mx, oracle, M, N, K, shift):
    """Pairs and single bytes with more columns than one round of workgroups covers, where the dispatcher goes by price: the few-row
    kernel and the one it takes."""
    rng = np.random.default_rng(M + K)
    a, b = random_operand(rng, M, K), random_operand(rng, N, K)
    da, db = [dev(a[0])] + [dev(t, shift) for t in a[1:]], [dev(b[0])] + [dev(t, shift) for t in b[1:]]
    for words in (True, False):
        want = oracle.gemm((a[0], a[1], a[2] if words else None), (b[0], b[1], b[2] if words else None))
        args = (da[0], da[1], da[2] if words else None, db[0], db[1], db[2] if words else None, "f32")
        close(mx.mx_gemm_mbs(*args), want, (M, N, K, words))
        with mx.forced(gemm_shape=5):
            close(mx.mx_gemm_mbs(*args), want, (M, N, K, words, "few rows"))


@pytest.mark.parametrize("K,shift", [(512, 0), (2880, 0), (2240, 1), (4096, 2), (96, 0)])
def test_grouped_few_rows(mx, oracle, K, shift):
    rng = np.random.default_rng(K + shift)
    sizes = [0, 1, 16, 17, 0, 32, 33, 70, 0, 3, 0, 0]
    G, N = len(sizes), 70
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    M = int(offsets[-1]) + 2  # two rows past the last group stay untouched
    assert M <= 32 * G
    a, b = random_operand(rng, M, K), random_operand(rng, G * N, K)
    da, db = [dev(a[0])] + [dev(t, shift) for t in a[1:]], [dev(b[0])] + [dev(t, shift) for t in b[1:]]
    off = torch.from_numpy(offsets).cuda()
    for mbs in (True, False):
        out = torch.full((M, N), -3.0, dtype=torch.float32, device="cuda")
        mx.mx_gemm_mbs_grouped(da[0], da[1], da[2] if mbs else None, db[0], db[1], db[2] if mbs else None, off, N, "f32", out=out)
        assert bool((out[M - 2:] == -3.0).all())
        for e in range(G):
            lo, hi = offsets[e], offsets[e + 1]
            if lo == hi:
                continue
            ra, rb = [t[lo:hi] for t in a], [t[e * N:(e + 1) * N] for t in b]
            if not mbs:
                ra[2] = rb[2] = None
            close(out[lo:hi], oracle.gemm(tuple(ra), tuple(rb)), (K, shift, mbs, e))


@pytest.mark.parametrize("K,shift", [(320, 0), (96, 1)])
@pytest.mark.parametrize("hot", [0, 63, 64, 129])
def test_grouped_few_rows_most_in_one_group(mx, oracle, K, shift, hot):
    """More groups than lanes, nearly all rows in one of them: its tile-rows are found behind and in front of empty groups."""
    rng = np.random.default_rng(K + hot)
    G, N = 130, 40
    sizes = np.where(np.arange(G) % 7 == 3, 1, 0)
    sizes[hot] = 16 * 45 + 1
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    M = int(offsets[-1])
    assert "few rows" in mx.gemm_plan(M, N, K, grouped=True, num_groups=G)
    a, b = random_operand(rng, M, K), random_operand(rng, G * N, K)
    da, db = [dev(a[0])] + [dev(t, shift) for t in a[1:]], [dev(b[0])] + [dev(t, shift) for t in b[1:]]
    out = mx.mx_gemm_mbs_grouped(*da, *db, torch.from_numpy(offsets).cuda(), N, "f32")
    for e in np.flatnonzero(sizes):
        lo, hi = offsets[e], offsets[e + 1]
        close(out[lo:hi], oracle.gemm(tuple(t[lo:hi] for t in a), tuple(t[e * N:(e + 1) * N] for t in b)), (K, hot, e))


# N: the kernel's one, two and four fragments of B; K: shares of one, two, three and four macro blocks per wavefront (the last
# wavefronts of some have fewer, or none), then a whole chunk and one, two and four of another
@pytest.mark.parametrize("M,N", [(17, 250), (33, 4113), (64, 8209), (32, 100), (16, 4100)])
@pytest.mark.parametrize("K", [512, 1024, 1536, 2560, 3072, 3584, 4096, 4608, 5120, 6656, 7680, 8192])
def test_fused_waits_for_weights_from_memory(mx, M, N, K):
    """mx_gemm_mbs_quantize_a bit for bit the quantizer and the GEMM, on weights that no cache holds any more: what a wait lets
    fly then has not arrived when it is read."""
    rng = np.random.default_rng(M + K)
    x = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)).cuda().to(torch.bfloat16)
    w = [dev(t) for t in random_operand(rng, N, K)]
    want = mx.mx_gemm_mbs(*mx.mx_quantize_mbs(x, "oas"), *w, "f32")
    evict = torch.empty(1 << 29, dtype=torch.uint8, device="cuda")
    for i in range(3):
        evict.fill_(i)
        got = mx.mx_gemm_mbs_quantize_a(x, "oas", *w, "f32")
        assert torch.equal(got, want), (M, N, K, i)
