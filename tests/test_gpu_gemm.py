"""GPU parity: scaled FP8 GEMM (NT / NN / TN) against the float64 oracle."""
import numpy as np
import pytest
import torch

from oracle import fp8, gemm, scaling
from paper_2505_20524_amd import fog, synth
from parity import check_bf16, check_gemm_elementwise, dev, fscalar, host_u16

pytestmark = pytest.mark.gpu


def lay(layout, A_mk, B_nk):
    if layout == gemm.NT:
        return A_mk, B_nk
    if layout == gemm.NN:
        return A_mk, np.ascontiguousarray(B_nk.T)
    return np.ascontiguousarray(A_mk.T), np.ascontiguousarray(B_nk.T)


def run_gemm(layout, A8, fa, sa, B8, fb, sb, M, N, K, ldc_pad=0):
    C = torch.full((M, N + ldc_pad), 0x7FC0, dtype=torch.int16, device="cuda")[:, :N] if ldc_pad else \
        torch.full((M, N), 0x7FC0, dtype=torch.int16, device="cuda")
    fog.fp8_gemm(layout, M, N, K, dev(A8), fa, fscalar(sa), dev(B8), fb, fscalar(sb), C)
    torch.cuda.synchronize()
    return host_u16(C)


def absdot(layout, a, fa, sa, b, fb, sb):
    """sinv_a sinv_b (|decode(A)| x |decode(B)|): the magnitude each output element accumulates."""
    A, B = np.abs(fp8.decode(a, fa)), np.abs(fp8.decode(b, fb))
    acc = A @ B.T if layout == gemm.NT else (A @ B if layout == gemm.NN else A.T @ B)
    return np.float64(sa) * np.float64(sb) * acc


def quantized_layer(seed, M, N, K, fa=fp8.E4M3, fb=fp8.E4M3):
    x, w, _ = synth.small_linear(seed, M, N, K)
    rx, rxi = scaling.compute_scale(scaling.amax(x), fa)
    rw, rwi = scaling.compute_scale(scaling.amax(w), fb)
    return scaling.quantize(x, rx, fa), rxi, scaling.quantize(w, rw, fb), rwi


SHAPES = [(512, 1024, 1024), (304, 528, 384), (272, 16, 144), (16, 272, 16), (1024, 512, 2048), (48, 48, 4096)]


@pytest.mark.parametrize("layout", [gemm.NT, gemm.NN, gemm.TN])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_gemm_parity(layout, M, N, K):
    A8, sa, B8, sb = quantized_layer(M + N + K, M, N, K)
    a, b = lay(layout, A8, B8)
    ref = gemm.fp8_gemm(layout, a, fp8.E4M3, sa, b, fp8.E4M3, sb)
    got = run_gemm(layout, a, fp8.E4M3, sa, b, fp8.E4M3, sb, M, N, K)
    stats = check_bf16(got, ref, what="gemm %d %dx%dx%d" % (layout, M, N, K))
    assert stats["max_steps"] <= 1
    # the tensor-normalised gate says little about elements far below the maximum (the x50 outlier channels make most
    # of them so): each element against its own value and its own accumulated magnitude
    check_gemm_elementwise(got, ref, absdot(layout, a, fp8.E4M3, sa, b, fp8.E4M3, sb), what="gemm %d %dx%dx%d" % (layout, M, N, K))


@pytest.mark.parametrize("layout", [gemm.NT, gemm.NN, gemm.TN])
def test_gemm_padded_leading_dimensions(layout):
    """Operands and result as views of wider buffers (lda, ldb, ldc larger than the rows): nothing outside the
    views is read into the result or written."""
    M, N, K = 304, 528, 400
    A8, sa, B8, sb = quantized_layer(77, M, N, K)
    a, b = lay(layout, A8, B8)
    ref = gemm.fp8_gemm(layout, a, fp8.E4M3, sa, b, fp8.E4M3, sb)
    pa, pb, pc = 16, 48, 8
    abuf = torch.full((a.shape[0], a.shape[1] + pa), 0x7E, dtype=torch.uint8, device="cuda")     # padding = largest code: a leak would show
    bbuf = torch.full((b.shape[0], b.shape[1] + pb), 0x7E, dtype=torch.uint8, device="cuda")
    abuf[:, :a.shape[1]] = dev(a)
    bbuf[:, :b.shape[1]] = dev(b)
    cbuf = torch.full((M, N + pc), 0x7FC0, dtype=torch.int16, device="cuda")
    fog.fp8_gemm(layout, M, N, K, abuf[:, :a.shape[1]], fp8.E4M3, fscalar(sa), bbuf[:, :b.shape[1]], fp8.E4M3, fscalar(sb), cbuf[:, :N])
    torch.cuda.synchronize()
    assert (cbuf[:, N:] == 0x7FC0).all()
    check_bf16(host_u16(cbuf[:, :N].contiguous()), ref, what="padded ld, layout %d" % layout)


def test_gemm_ragged_rows_nt():
    """NT takes any M and N (rows of the operands); K only has to be a multiple of 16."""
    for (M, N, K) in [(1, 1, 16), (257, 259, 160), (300, 37, 128), (5, 700, 400)]:
        A8, sa, B8, sb = quantized_layer(M * 7 + N, M, N, K)
        ref = gemm.fp8_gemm(gemm.NT, A8, fp8.E4M3, sa, B8, fp8.E4M3, sb)
        got = run_gemm(gemm.NT, A8, fp8.E4M3, sa, B8, fp8.E4M3, sb, M, N, K, ldc_pad=(3 if N % 2 else 0))
        check_bf16(got, ref, what="ragged %dx%dx%d" % (M, N, K))


@pytest.mark.parametrize("layout", [gemm.NT, gemm.NN, gemm.TN])
@pytest.mark.parametrize("fa,fb", [(fp8.E5M2, fp8.E4M3), (fp8.E4M3, fp8.E5M2), (fp8.E5M2, fp8.E5M2)])
def test_gemm_mixed_formats(layout, fa, fb):
    M, N, K = 320, 288, 256
    A8, sa, B8, sb = quantized_layer(17, M, N, K, fa, fb)
    a, b = lay(layout, A8, B8)
    ref = gemm.fp8_gemm(layout, a, fa, sa, b, fb, sb)
    got = run_gemm(layout, a, fa, sa, b, fb, sb, M, N, K)
    check_bf16(got, ref, what="formats")
    check_gemm_elementwise(got, ref, absdot(layout, a, fa, sa, b, fb, sb), what="formats")


@pytest.mark.parametrize("layout", [gemm.NT, gemm.NN, gemm.TN])
def test_gemm_exact_cases(layout):
    """Small integers with power-of-two scales: the result is exact and bf16-representable."""
    rng = np.random.default_rng(5)
    M, N, K = 288, 272, 256
    Ai = rng.integers(-2, 3, size=(M, K)); Bi = rng.integers(-2, 3, size=(N, K))
    Ai[rng.random((M, K)) < 0.7] = 0; Bi[rng.random((N, K)) < 0.7] = 0      # keep |sums| < 256: exact in bf16
    A8 = scaling.quantize(synth.f32_to_bf16_bits(Ai.astype(np.float32)), np.float32(1), fp8.E4M3)
    B8 = scaling.quantize(synth.f32_to_bf16_bits(Bi.astype(np.float32)), np.float32(1), fp8.E5M2)
    a, b = lay(layout, A8, B8)
    got = run_gemm(layout, a, fp8.E4M3, 0.5, b, fp8.E5M2, 0.25, M, N, K)
    want = (Ai @ Bi.T) / 8.0
    assert np.abs(Ai @ Bi.T).max() < 256
    assert np.array_equal(synth.bf16_bits_to_f32(got).astype(np.float64), want)
    # one-hot operands: a single non-zero at a known place
    A1 = np.zeros((M, K), np.uint8); B1 = np.zeros((N, K), np.uint8)
    A1[200, 77] = 0x40; B1[131, 77] = 0x44
    a, b = lay(layout, A1, B1)
    got = synth.bf16_bits_to_f32(run_gemm(layout, a, fp8.E4M3, 1.0, b, fp8.E4M3, 1.0, M, N, K))
    want = np.zeros((M, N), np.float32); want[200, 131] = 6.0
    assert np.array_equal(got, want)


def test_gemm_k_zero_and_empty():
    C = torch.full((32, 48), 0x7FC0, dtype=torch.int16, device="cuda")
    one = fscalar(1.0)
    lib = fog.load()
    st = torch.cuda.current_stream().cuda_stream
    assert lib.fog_fp8_gemm(0, 32, 48, 0, None, 0, 0, one.data_ptr(), None, 0, 0, one.data_ptr(), C.data_ptr(), 48, None, 0, st) == 0
    torch.cuda.synchronize()
    assert (C.cpu().numpy() == 0).all()
    assert lib.fog_fp8_gemm(0, 0, 48, 16, None, 0, 16, one.data_ptr(), None, 0, 16, one.data_ptr(), C.data_ptr(), 48, None, 0, st) == 0


def test_gemm_argument_errors():
    lib = fog.load()
    st = torch.cuda.current_stream().cuda_stream
    A = torch.zeros(64 * 64, dtype=torch.uint8, device="cuda")
    C = torch.zeros(64 * 64, dtype=torch.int16, device="cuda")
    one = fscalar(1.0)
    p, o = A.data_ptr(), one.data_ptr()
    assert lib.fog_fp8_gemm(0, 64, 64, 64, None, 0, 64, o, p, 0, 64, o, C.data_ptr(), 64, None, 0, st) == 1
    assert lib.fog_fp8_gemm(0, 64, 64, 64, p, 0, 32, o, p, 0, 64, o, C.data_ptr(), 64, None, 0, st) == 2
    assert lib.fog_fp8_gemm(0, 64, 64, 64, p + 1, 0, 64, o, p, 0, 64, o, C.data_ptr(), 64, None, 0, st) == 3
    assert lib.fog_fp8_gemm(0, 64, 64, 40, p, 0, 48, o, p, 0, 48, o, C.data_ptr(), 64, None, 0, st) == 4
    assert lib.fog_fp8_gemm(1, 64, 40, 64, p, 0, 64, o, p, 0, 48, o, C.data_ptr(), 64, None, 0, st) == 4
    assert lib.fog_fp8_gemm(5, 64, 64, 64, p, 0, 64, o, p, 0, 64, o, C.data_ptr(), 64, None, 0, st) == 4
    assert lib.fog_fp8_gemm(0, -1, 64, 64, p, 0, 64, o, p, 0, 64, o, C.data_ptr(), 64, None, 0, st) == 2


def test_config2_full_size_all_three_products():
    """Config 2 whole (tokens 4096, in 2048, out 8192): forward, data gradient, weight gradient,
    each both in its native layout and as NT on the transposed copies the cast kernel emits."""
    cfg = synth.CONFIGS[2]
    t = synth.linear_tensors(cfg, 0)
    M, N, K = 4096, 8192, 2048
    dv = {}
    ora = {}
    for name, fmt in (("X", fp8.E4M3), ("W", fp8.E4M3), ("dY", fp8.E5M2)):
        xb = t[name]
        xd = dev(xb)
        am, s, si = (torch.zeros(1, device="cuda") for _ in range(3))
        fog.amax(xd, am); fog.scale(am, fmt, s, si)
        q = torch.zeros(xb.shape, dtype=torch.uint8, device="cuda")
        qT = torch.zeros(xb.shape[::-1], dtype=torch.uint8, device="cuda")
        fog.quantize(xd, fmt, s, q=q, qT=qT)
        rho, rinv = scaling.compute_scale(scaling.amax(xb), fmt)
        want = scaling.quantize(xb, rho, fmt)
        assert np.float32(si.item()) == rinv
        assert np.array_equal(q.cpu().numpy(), want) and np.array_equal(qT.cpu().numpy(), want.T)
        dv[name] = (q, qT, si)
        ora[name] = (want, rinv)

    def gpu(layout, m, n, k, A, fa, sa, B, fb, sb):
        C = torch.zeros((m, n), dtype=torch.int16, device="cuda")
        fog.fp8_gemm(layout, m, n, k, A, fa, sa, B, fb, sb, C)
        torch.cuda.synchronize()
        return host_u16(C)

    X, W, dY = ora["X"], ora["W"], ora["dY"]
    ref = gemm.fp8_gemm(gemm.NT, X[0], fp8.E4M3, X[1], W[0], fp8.E4M3, W[1])                     # Y = X W^T
    check_bf16(gpu(fog.NT, M, N, K, dv["X"][0], 0, dv["X"][2], dv["W"][0], 0, dv["W"][2]), ref, what="fwd")
    ref = gemm.fp8_gemm(gemm.NN, dY[0], fp8.E5M2, dY[1], W[0], fp8.E4M3, W[1])                   # dX = dY W
    check_bf16(gpu(fog.NN, M, K, N, dv["dY"][0], 1, dv["dY"][2], dv["W"][0], 0, dv["W"][2]), ref, what="dgrad NN")
    check_bf16(gpu(fog.NT, M, K, N, dv["dY"][0], 1, dv["dY"][2], dv["W"][1], 0, dv["W"][2]), ref, what="dgrad NT(W^T)")
    ref = gemm.fp8_gemm(gemm.TN, dY[0], fp8.E5M2, dY[1], X[0], fp8.E4M3, X[1])                   # dW = dY^T X
    check_bf16(gpu(fog.TN, N, K, M, dv["dY"][0], 1, dv["dY"][2], dv["X"][0], 0, dv["X"][2]), ref, what="wgrad TN")
    check_bf16(gpu(fog.NT, N, K, M, dv["dY"][1], 1, dv["dY"][2], dv["X"][1], 0, dv["X"][2]), ref, what="wgrad NT(dY^T, X^T)")


def run_gemm_ws(layout, a, fa, sa, b, fb, sb, M, N, K, ws_bytes=None):
    """fog_fp8_gemm with the workspace the query asks for (or `ws_bytes`); returns (C bits, bytes the query asked for)."""
    need = fog.fp8_gemm_workspace(layout, M, N, K)
    n = need if ws_bytes is None else ws_bytes
    ws = torch.full((max(n, 16),), 0xFF, dtype=torch.uint8, device="cuda") if n else None      # NaN patterns: a partial read before written would show
    C = torch.full((M, N), 0x7FC0, dtype=torch.int16, device="cuda")
    fog.fp8_gemm(layout, M, N, K, dev(a), fa, fscalar(sa), dev(b), fb, fscalar(sb), C, workspace=ws)
    torch.cuda.synchronize()
    return host_u16(C), need


SPLIT_SHAPES = [   # few output tiles, long contraction: the query names room on all of them, five are split (PLANNED_SPLITS names the kernels)
    (gemm.TN, 2048, 2048, 16384),     # config 4: weight gradient of the output projection (64 tiles)
    (gemm.NN, 4096, 2048, 8192),      # config 2: data gradient (128 tiles)
    (gemm.NT, 256, 256, 32768),       # one tile
    (gemm.NN, 1024, 1024, 8192),      # 16 tiles
    (gemm.NT, 300, 200, 5008),        # ragged edges, contraction not a multiple of the chunk or of a K-step
    (gemm.TN, 272, 528, 4112),        # K-major operands with a ragged contraction
    (gemm.NN, 48, 1040, 12304),
]


@pytest.mark.parametrize("layout,M,N,K", SPLIT_SHAPES)
def test_gemm_contraction_split(layout, M, N, K):
    """With the workspace the query asks for, launches of few tiles are cut along the contraction (binary32 partial
    tiles, reduced in a fixed order): same gate as the unsplit kernel, the same bits on a second call, and without a
    workspace (or with one that is too small) the unsplit kernel answers inside the same gate."""
    fa, fb = (fp8.E5M2, fp8.E4M3) if layout != gemm.NT else (fp8.E4M3, fp8.E4M3)
    A8, sa, B8, sb = quantized_layer(M + 3 * N + K, M, N, K, fa, fb)
    a, b = lay(layout, A8, B8)
    ref = gemm.fp8_gemm(layout, a, fa, sa, b, fb, sb)
    got, need = run_gemm_ws(layout, a, fa, sa, b, fb, sb, M, N, K)
    assert need > 0 and need % (256 * 256 * 4) == 0, "the query did not ask for a split on this shape"
    st = check_bf16(got, ref, what="split %d %dx%dx%d" % (layout, M, N, K))
    assert st["max_steps"] <= 1
    check_gemm_elementwise(got, ref, absdot(layout, a, fa, sa, b, fb, sb), what="split %d %dx%dx%d" % (layout, M, N, K))
    again, _ = run_gemm_ws(layout, a, fa, sa, b, fb, sb, M, N, K)
    assert np.array_equal(got, again)                      # deterministic: no atomics, fixed order of the chunks
    for small in (0, need - 1):
        unsplit, _ = run_gemm_ws(layout, a, fa, sa, b, fb, sb, M, N, K, ws_bytes=small)
        check_bf16(unsplit, ref, what="unsplit fallback")
    # the two routes differ only in the order of binary32 additions: at most one bf16 step, on few elements
    steps = np.abs(got.astype(np.int32) - unsplit.astype(np.int32))
    assert steps.max() <= 1 and (steps > 0).mean() < 0.05


def test_gemm_split_exact_integers_and_query():
    """Small integers: every partial sum is exact, so split and unsplit give identical, exact results; shapes with
    enough tiles ask for no workspace."""
    rng = np.random.default_rng(11)
    M, N, K = 256, 512, 16384
    Ai = rng.integers(-2, 3, size=(M, K)); Bi = rng.integers(-2, 3, size=(N, K))
    Ai[rng.random((M, K)) < 0.97] = 0; Bi[rng.random((N, K)) < 0.9] = 0
    assert np.abs(Ai @ Bi.T).max() < 256
    A8 = scaling.quantize(synth.f32_to_bf16_bits(Ai.astype(np.float32)), np.float32(1), fp8.E4M3)
    B8 = scaling.quantize(synth.f32_to_bf16_bits(Bi.astype(np.float32)), np.float32(1), fp8.E4M3)
    got, need = run_gemm_ws(gemm.NT, A8, fp8.E4M3, 0.5, B8, fp8.E4M3, 0.5, M, N, K)
    assert need > 0
    assert np.array_equal(synth.bf16_bits_to_f32(got).astype(np.float64), (Ai @ Bi.T) / 4.0)
    for (layout, m, n, k) in [(gemm.NT, 8192, 12288, 4096), (gemm.TN, 14336, 4096, 8192), (gemm.NT, 512, 1024, 1024)]:
        assert fog.fp8_gemm_workspace(layout, m, n, k) == 0


TILE_SHAPES = [   # (layout, M, N, K, padding of C's rows, tile, workgroups per CU): products of few 256 x 256 tiles, each smaller tile per layout
    (gemm.NT, 65, 63, 16, 1, 64, 64, 2), (gemm.NT, 500, 776, 1040, 8, 64, 64, 2), (gemm.NN, 129, 80, 272, 3, 64, 64, 2), (gemm.TN, 64, 144, 5, 0, 64, 64, 2),
    (gemm.NT, 1900, 1500, 3088, 8, 128, 128, 1), (gemm.NN, 1777, 2064, 3088, 0, 128, 128, 1), (gemm.TN, 1296, 1040, 2001, 5, 128, 128, 1),
    (gemm.NT, 7900, 1184, 384, 0, 128, 128, 2), (gemm.NN, 2050, 3216, 144, 8, 128, 128, 2), (gemm.TN, 6336, 1104, 155, 0, 128, 128, 2),
    (gemm.NT, 1777, 3088, 2064, 0, 256, 128, 1), (gemm.NN, 4000, 1808, 2064, 3, 256, 128, 1), (gemm.TN, 3088, 2064, 1777, 8, 256, 128, 1),
]


@pytest.mark.parametrize("layout,M,N,K,pad,tile_m,tile_n,per_cu", TILE_SHAPES)
def test_gemm_small_tiles(layout, M, N, K, pad, tile_m, tile_n, per_cu):
    """Products whose 256 x 256 tiles would leave most of the chip idle run on smaller tiles: edges of the tiles, contractions
    that end inside a stage, padded and unaligned C, against the oracle; nothing outside C's rows is written."""
    assert fog.probe_gemm_plan(layout, M, N, K)[:4] == (tile_m, tile_n, per_cu, 1), "another kernel runs on this shape"
    fa, fb = (fp8.E5M2, fp8.E4M3) if layout != gemm.NT else (fp8.E4M3, fp8.E4M3)
    A8, sa, B8, sb = quantized_layer(M + 5 * N + K, M, N, K, fa, fb)
    a, b = lay(layout, A8, B8)
    ref = gemm.fp8_gemm(layout, a, fa, sa, b, fb, sb)
    store = torch.full((M + 1, N + pad), 0x7FC0, dtype=torch.int16, device="cuda")
    C = store[:M, :N]
    fog.fp8_gemm(layout, M, N, K, dev(a), fa, fscalar(sa), dev(b), fb, fscalar(sb), C)
    torch.cuda.synchronize()
    got = host_u16(store)
    assert (got[M] == 0x7FC0).all() and (got[:, N:] == 0x7FC0).all()
    what = "tiles %d %dx%dx%d" % (layout, M, N, K)
    check_bf16(got[:M, :N], ref, what=what)
    check_gemm_elementwise(got[:M, :N], ref, absdot(layout, a, fa, sa, b, fb, sb), what=what)


@pytest.mark.parametrize("layout,M,N,K", [(gemm.NT, 66, 1936, 9520), (gemm.NN, 80, 368, 11520), (gemm.TN, 304, 272, 8200), (gemm.NT, 328, 1584, 6000),
                                          (gemm.NN, 2339, 400, 9616)])
def test_gemm_small_tile_split(layout, M, N, K):
    """With room for a split on smaller tiles (the fourth shape is left whole all the same): partial tiles that reach past C, a last chunk
    shorter than the others, the workspace full of NaN patterns beforehand and its end untouched; the same bits on a second call."""
    fa, fb = (fp8.E5M2, fp8.E4M3) if layout != gemm.NT else (fp8.E4M3, fp8.E4M3)
    A8, sa, B8, sb = quantized_layer(M + 7 * N + K, M, N, K, fa, fb)
    a, b = lay(layout, A8, B8)
    ref = gemm.fp8_gemm(layout, a, fa, sa, b, fb, sb)
    need = fog.fp8_gemm_workspace(layout, M, N, K)
    assert need > 0
    got = []
    for _ in range(2):
        store = torch.full((need + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
        C = torch.full((M, N), 0x7FC0, dtype=torch.int16, device="cuda")
        fog.fp8_gemm(layout, M, N, K, dev(a), fa, fscalar(sa), dev(b), fb, fscalar(sb), C, workspace=store[:need])
        torch.cuda.synchronize()
        assert (store[need:] == 0xFF).all()
        got.append(host_u16(C))
    assert np.array_equal(got[0], got[1])
    what = "split tiles %d %dx%dx%d" % (layout, M, N, K)
    check_bf16(got[0], ref, what=what)
    check_gemm_elementwise(got[0], ref, absdot(layout, a, fa, sa, b, fb, sb), what=what)


def wide(a, pad):
    """The matrix as a view of a wider buffer whose padding holds 0x7E (the largest E4M3 code, a NaN in E5M2): a leak would show."""
    buf = torch.full((a.shape[0], a.shape[1] + pad), 0x7E, dtype=torch.uint8, device="cuda")
    buf[:, :a.shape[1]] = dev(a)
    return buf[:, :a.shape[1]]


E4, E5 = fp8.E4M3, fp8.E5M2
BIG_EDGE_SHAPES = [   # (layout, M, N, K, formats, padding of A's, B's and C's rows): 256 x 256 tiles, one and two rounds of them
    (gemm.NT, 911, 8860, 432, E4, E5, 16, 0, 0),          # C's rows allow no 16-byte store (8860 = 4 mod 8)
    (gemm.NT, 5889, 4104, 400, E5, E5, 0, 48, 8),
    (gemm.NN, 2706, 3376, 400, E5, E4, 48, 16, 3),
    (gemm.NN, 6935, 3504, 400, E4, E5, 16, 0, 0),
    (gemm.TN, 5296, 1712, 390, E5, E5, 0, 16, 8),
    (gemm.TN, 6704, 3648, 385, E4, E4, 32, 16, 5),
]


@pytest.mark.parametrize("layout,M,N,K,fa,fb,pa,pb,pc", BIG_EDGE_SHAPES)
def test_gemm_big_tile_edges(layout, M, N, K, fa, fb, pa, pb, pc):
    """The 256 x 256 kernel away from its home ground: edge tiles in both directions, contractions that end inside a K-step,
    padded operands, padded and unaligned C, the format pairs; nothing outside C's rows is written."""
    assert fog.probe_gemm_plan(layout, M, N, K)[:4] == (256, 256, 1, 1), "another kernel runs on this shape"
    A8, sa, B8, sb = quantized_layer(M + 11 * N + K, M, N, K, fa, fb)
    a, b = lay(layout, A8, B8)
    ref = gemm.fp8_gemm(layout, a, fa, sa, b, fb, sb)
    store = torch.full((M + 1, N + pc), 0x7FC0, dtype=torch.int16, device="cuda")
    fog.fp8_gemm(layout, M, N, K, wide(a, pa), fa, fscalar(sa), wide(b, pb), fb, fscalar(sb), store[:M, :N])
    torch.cuda.synchronize()
    got = host_u16(store)
    assert (got[M] == 0x7FC0).all() and (got[:, N:] == 0x7FC0).all()
    what = "edges %d %dx%dx%d" % (layout, M, N, K)
    check_bf16(got[:M, :N], ref, what=what)
    check_gemm_elementwise(got[:M, :N], ref, absdot(layout, a, fa, sa, b, fb, sb), what=what)


PLANNED_SPLITS = [   # (layout, M, N, K, formats, padding of C's rows, tile): every kernel that splits, per layout, ragged
    (gemm.NT, 73, 77, 4848, E4, E4, 3, 64, 64), (gemm.NN, 87, 112, 4592, E5, E4, 0, 64, 64), (gemm.TN, 64, 80, 4909, E4, E5, 8, 64, 64),
    (gemm.NT, 2321, 65, 12608, E5, E4, 7, 128, 128), (gemm.NN, 69, 1168, 13456, E4, E5, 8, 128, 128), (gemm.TN, 80, 1392, 6508, E5, E5, 0, 128, 128),
    (gemm.NT, 5987, 136, 7472, E4, E4, 8, 256, 128), (gemm.NN, 130, 5552, 7664, E5, E5, 1, 256, 128), (gemm.TN, 8592, 80, 10583, E5, E4, 0, 256, 128),
    (gemm.NT, 8274, 136, 12480, E4, E5, 0, 256, 256), (gemm.NN, 1744, 2480, 9296, E5, E4, 5, 256, 256), (gemm.TN, 6432, 144, 13908, E5, E4, 8, 256, 256),
]


@pytest.mark.parametrize("layout,M,N,K,fa,fb,pc,tile_m,tile_n", PLANNED_SPLITS)
def test_gemm_split_kernels(layout, M, N, K, fa, fb, pc, tile_m, tile_n):
    """The contraction split on each tile, partial tiles that reach past C, a shorter last chunk: the workspace is full of NaN patterns
    beforehand, is used, and its end is not touched; nothing outside C's rows is written; the same bits on a second call."""
    plan = fog.probe_gemm_plan(layout, M, N, K, True)
    assert plan[:2] == (tile_m, tile_n) and plan[3] > 1, "another kernel runs on this shape"
    assert K % plan[4] != 0
    A8, sa, B8, sb = quantized_layer(M + 13 * N + K, M, N, K, fa, fb)
    a, b = lay(layout, A8, B8)
    ref = gemm.fp8_gemm(layout, a, fa, sa, b, fb, sb)
    need = fog.fp8_gemm_workspace(layout, M, N, K)
    used = plan[3] * -(-M // tile_m) * -(-N // tile_n) * tile_m * tile_n * 4
    assert 0 < used <= need
    got = []
    for _ in range(2):
        ws = torch.full((need + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
        store = torch.full((M + 1, N + pc), 0x7FC0, dtype=torch.int16, device="cuda")
        fog.fp8_gemm(layout, M, N, K, dev(a), fa, fscalar(sa), dev(b), fb, fscalar(sb), store[:M, :N], workspace=ws[:need])
        torch.cuda.synchronize()
        assert not (ws[:used].view(torch.int32) == -1).any() and (ws[used:] == 0xFF).all()
        got.append(host_u16(store))
    assert np.array_equal(got[0], got[1])
    assert (got[0][M] == 0x7FC0).all() and (got[0][:, N:] == 0x7FC0).all()
    what = "split %dx%d %d %dx%dx%d" % (tile_m, tile_n, layout, M, N, K)
    check_bf16(got[0][:M, :N], ref, what=what)
    check_gemm_elementwise(got[0][:M, :N], ref, absdot(layout, a, fa, sa, b, fb, sb), what=what)
