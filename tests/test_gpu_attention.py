"""GPU parity: FP8 attention forward / backward against the float64 oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import attention, bf16, fp8, scaling
from paper_2505_20524_amd import fog, synth
import mfma_model
from parity import check_attention, check_bf16, dev, fscalar, host_u16

pytestmark = pytest.mark.gpu

SAMPLED_EXCEED = 0.06     # a sample of 18 rows, a third of them short (0, 1, 63, 64, ...): one short row may move whole (measured: none did)


def cast_all(q, k, v, do):
    out = {}
    for name, t, fmt in (("q", q, fp8.E4M3), ("k", k, fp8.E4M3), ("v", v, fp8.E4M3), ("do", do, fp8.E5M2)):
        rho, rinv = scaling.compute_scale(scaling.amax(t), fmt)
        out[name] = (scaling.quantize(t.reshape(-1, t.shape[-1]), rho, fmt).reshape(t.shape), rinv)
    return out


def kv_of(c, h):
    """Key/value head of query head h: the tensors of c["k"], c["v"] are [B, H_kv, S, D] (H_kv == H: multi-head)."""
    H, Hkv = c["q"][0].shape[1], c["k"][0].shape[1]
    return h // (H // Hkv)


def gpu_fwd(c, B, H, S, s, causal, want_amax=True, rho_p=448.0):
    O = torch.full((B, H, S, 128), 0x7FC0, dtype=torch.int16, device="cuda")
    lse = torch.full((B, H, S), float("nan"), device="cuda")
    am = torch.full((1,), -1.0, device="cuda") if want_amax else None
    fog.fp8_attn_fwd(B, H, S, 128, s, causal, dev(c["q"][0]), dev(c["k"][0]), dev(c["v"][0]),
                     fscalar(c["q"][1]), fscalar(c["k"][1]), fscalar(c["v"][1]), fscalar(rho_p), O, lse, amax_p=am,
                     H_kv=c["k"][0].shape[1])
    torch.cuda.synchronize()
    return host_u16(O), lse.cpu().numpy(), (am.item() if want_amax else None)


def oracle_fwd_heads(c, heads, s, causal, rho_p=448.0):
    res = {}
    for (b, h) in heads:
        hk = kv_of(c, h)
        res[(b, h)] = attention.attn_fwd_head(c["q"][0][b, h], c["k"][0][b, hk], c["v"][0][b, hk],
                                              c["q"][1], c["k"][1], c["v"][1], s, rho_p, causal)
    return res


def check_fwd(c, B, H, S, s, causal, heads, rho_p=448.0):
    O, lse, am = gpu_fwd(c, B, H, S, s, causal, rho_p=rho_p)
    rho_p = min(rho_p, 448.0)            # the forward uses a probability scale above the format's maximum as 448
    ref = oracle_fwd_heads(c, heads, s, causal, rho_p)
    pmax = 0.0
    for (b, h), (Or, lr, ap) in ref.items():
        hk = kv_of(c, h)
        dx = mfma_model.logit_uncertainty(c["q"][0][b, h], c["k"][0][b, hk], c["q"][1], c["k"][1], s, causal)
        slack = mfma_model.fwd_cast_slack(c["q"][0][b, h], c["k"][0][b, hk], c["v"][0][b, hk], c["q"][1], c["k"][1], c["v"][1],
                                         s, rho_p, causal, dx=dx)
        check_attention(O[b, h], Or, slack, what="O[%d,%d]" % (b, h))
        lunc = mfma_model.lse_uncertainty(c["q"][0][b, h], c["k"][0][b, hk], c["q"][1], c["k"][1], s, causal, dx=dx)
        assert np.all(np.abs(lse[b, h] - lr) <= 2e-4 + lunc), "lse"
        pmax = max(pmax, float(ap))
    assert np.isfinite(lse).all()
    if len(heads) == B * H:
        assert abs(am - pmax) <= 1e-4 * pmax
    assert 0.5 < am <= 1.0 + 1e-6
    return O, lse


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,H,S", [(1, 1, 64), (1, 2, 128), (2, 2, 320), (1, 3, 576)])
def test_forward_parity(B, H, S, causal):
    q, k, v, do = synth.small_attention(1000 + S, B, H, S)
    c = cast_all(q, k, v, do)
    check_fwd(c, B, H, S, 1 / math.sqrt(128), causal, [(b, h) for b in range(B) for h in range(H)])


@pytest.mark.parametrize("rho_p", [100.0, 1000.0, 3000.0])
def test_probability_scale_other_than_the_format_maximum(rho_p):
    """scale_p below 448 wastes range.  Above 448 the forward uses 448 (p is taken against the running row reference
    there, so saturation would depend on the visiting order); the backward casts the normalised P, for which
    saturation is well defined (P > 448 / scale_p maps to 448), and takes its saturating-cast loops."""
    B, H, S = 1, 2, 256
    q, k, v, do = synth.small_attention(500 + int(rho_p), B, H, S)
    c = cast_all(q, k, v, do)
    heads = [(0, 0), (0, 1)]
    check_fwd(c, B, H, S, 0.125, True, heads, rho_p=rho_p)
    run_bwd(c, B, H, S, 0.125, True, heads, do, rho_p=rho_p)


def test_forward_fog_softmax_scale_and_q_zero():
    B, H, S = 1, 2, 256
    q, k, v, do = synth.small_attention(77, B, H, S)
    c = cast_all(q, k, v, do)
    check_fwd(c, B, H, S, 0.125, True, [(0, 0), (0, 1)])         # FOG's s = gamma_0^2 / sqrt(D) at D = 128
    # Q = 0: every p is 1 and P~ = 448 exactly, so O_i is the running mean of the decoded V rows
    c["q"] = (np.zeros_like(c["q"][0]), np.float32(1.0))
    O, lse, _ = gpu_fwd(c, B, H, S, 0.125, True)
    for h in range(H):
        vv = fp8.decode(c["v"][0][0, h], fp8.E4M3) * np.float64(c["v"][1])
        run = np.cumsum(vv, axis=0) / np.arange(1, S + 1)[:, None]
        check_bf16(O[0, h], run, rel=1e-5, what="running mean")
        assert np.abs(lse[0, h] - np.log2(np.arange(1, S + 1))).max() < 1e-5


def run_bwd(c, B, H, S, s, causal, heads, do_bits, rho_p=448.0, ds_scale_factor=1.0):
    """Feeds the ORACLE's forward results (O rounded to bf16, lse rounded to binary32) to both sides.
    Under grouped-query attention dK and dV of a key/value head are checked when all the query heads of
    its group are in `heads`: the oracle's per-head contributions are summed in float64 (the kernel sums
    them in binary32 before its one rounding), and so are the slacks of the cast decisions."""
    Hkv = c["k"][0].shape[1]
    G = H // Hkv
    O_bits = np.zeros((B, H, S, 128), np.uint16)
    lse = np.zeros((B, H, S), np.float32)

    def head_args(b, h):
        hk = h // G
        return (c["q"][0][b, h], c["k"][0][b, hk], c["v"][0][b, hk], c["q"][1], c["k"][1], c["v"][1])

    for (b, h) in heads:
        Or, lr, _ = attention.attn_fwd_head(*head_args(b, h), s, rho_p, causal)
        O_bits[b, h] = bf16.f64_to_bits_rne(Or)
        lse[b, h] = lr.astype(np.float32)
    # calibrate rho_dS from one oracle pass without the dS cast (delayed-style scale)
    amax_ds = 0.0
    for (b, h) in heads:
        r = attention.attn_bwd_head(*head_args(b, h), O_bits[b, h], do_bits[b, h], c["do"][0][b, h], c["do"][1], lse[b, h],
                                    s, rho_p, 1.0, causal, True, False)
        amax_ds = max(amax_ds, float(r[3]))
    rho_ds, _ = scaling.compute_scale(np.float32(amax_ds), fp8.E5M2)
    rho_ds = np.float32(rho_ds * ds_scale_factor)     # > 1: a stale (delayed) scale, the largest dS saturate
    dQ = torch.full((B, H, S, 128), 0x7FC0, dtype=torch.int16, device="cuda")
    dK, dV = (torch.full((B, Hkv, S, 128), 0x7FC0, dtype=torch.int16, device="cuda") for _ in range(2))
    am = torch.full((1,), -1.0, device="cuda")
    ws = torch.empty(fog.fp8_attn_workspace(B, H, S, 128, True, H_kv=Hkv), dtype=torch.uint8, device="cuda")
    fog.fp8_attn_bwd(B, H, S, 128, s, causal, dev(c["q"][0]), dev(c["k"][0]), dev(c["v"][0]),
                     fscalar(c["q"][1]), fscalar(c["k"][1]), fscalar(c["v"][1]), dev(O_bits), dev(do_bits), dev(c["do"][0]),
                     fscalar(c["do"][1]), dev(lse), fscalar(rho_p), fscalar(rho_ds), dQ, dK, dV, amax_ds=am, workspace=ws,
                     H_kv=Hkv)
    torch.cuda.synchronize()
    dQ, dK, dV = host_u16(dQ), host_u16(dK), host_u16(dV)
    group = {}
    for (b, h) in heads:
        tail = (O_bits[b, h], do_bits[b, h], c["do"][0][b, h], c["do"][1], lse[b, h], s, rho_p, rho_ds, causal)
        r = attention.attn_bwd_head(*head_args(b, h), *tail)
        sl = mfma_model.bwd_cast_slack(*head_args(b, h), *tail)
        check_attention(dQ[b, h], r[0], sl[0], what="dQ[%d,%d]" % (b, h))
        acc = group.setdefault((b, h // G), [0, 0.0, 0.0, 0.0, 0.0])
        acc[0] += 1
        acc[1] = acc[1] + r[1]; acc[2] = acc[2] + r[2]; acc[3] = acc[3] + sl[1]; acc[4] = acc[4] + sl[2]
    checked = 0
    for (b, hk), (n, dk, dv, sk, sv) in group.items():
        if n != G:
            continue            # not every query head of the group was evaluated
        check_attention(dK[b, hk], dk, sk, what="dK[%d,%d]" % (b, hk))
        check_attention(dV[b, hk], dv, sv, what="dV[%d,%d]" % (b, hk))
        checked += 1
    assert checked > 0
    if len(heads) == B * H:
        assert abs(am.item() - amax_ds) <= 1e-4 * amax_ds
    return dQ, dK, dV


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,H,S", [(1, 1, 64), (1, 2, 128), (2, 2, 320), (1, 2, 576)])
def test_backward_parity(B, H, S, causal):
    q, k, v, do = synth.small_attention(2000 + S, B, H, S)
    c = cast_all(q, k, v, do)
    run_bwd(c, B, H, S, 1 / math.sqrt(128), causal, [(b, h) for b in range(B) for h in range(H)], do)


@pytest.mark.parametrize("factor", [4.0, 64.0])
def test_backward_with_a_stale_ds_scale_saturates_like_the_oracle(factor):
    """A scale of dS several times too large (delayed scaling after the gradients grew): rho_ds dS exceeds the largest
    finite E5M2 value in some key blocks and not in others, so both the clamped and the unclamped form of the cast run."""
    B, H, S = 1, 2, 320
    q, k, v, do = synth.small_attention(2600 + int(factor), B, H, S)
    c = cast_all(q, k, v, do)
    run_bwd(c, B, H, S, 1 / math.sqrt(128), True, [(b, h) for b in range(B) for h in range(H)], do, ds_scale_factor=factor)


@pytest.mark.parametrize("causal", [True, False])
def test_backward_with_a_scale_beyond_any_gradient(causal):
    """A scale of dS so large (above 1e18) that rho_ds dS may leave binary32: the dK/dV kernel clamps infinities too before its
    casts.  Every dS that is not tiny saturates, in the oracle too."""
    B, H, S = 1, 2, 192
    q, k, v, do = synth.small_attention(2700, B, H, S)
    c = cast_all(q, k, v, do)
    run_bwd(c, B, H, S, 1 / math.sqrt(128), causal, [(b, h) for b in range(B) for h in range(H)], do, ds_scale_factor=2.0 ** 50)


@pytest.mark.parametrize("causal", [True, False])
def test_backward_with_an_infinite_output_gradient(causal):
    """One element of the bf16 dO is infinite (its code is saturated, as a cast under a delayed scale leaves it): D of that row is
    infinite and every dS of the row saturates at the largest finite code, exactly as it does for a huge finite element.
    dK and dV have to be the same bytes in the two cases."""
    B, H, S = 1, 2, 192
    q, k, v, do = synth.small_attention(2710, B, H, S)
    c = cast_all(q, k, v, do)
    s = 1 / math.sqrt(128)
    O, lse, _ = gpu_fwd(c, B, H, S, s, causal, want_amax=False)
    out = []
    for bits in (0x7F80, 0x7149):                  # +infinity, 1e30
        d = do.copy()
        d[0, 0, 100, 5] = bits
        dQ, dK, dV = (torch.full((B, H, S, 128), 0x7FC0, dtype=torch.int16, device="cuda") for _ in range(3))
        ws = torch.empty(fog.fp8_attn_workspace(B, H, S, 128, True), dtype=torch.uint8, device="cuda")
        fog.fp8_attn_bwd(B, H, S, 128, s, causal, dev(c["q"][0]), dev(c["k"][0]), dev(c["v"][0]),
                         fscalar(c["q"][1]), fscalar(c["k"][1]), fscalar(c["v"][1]), dev(O), dev(d), dev(c["do"][0]),
                         fscalar(c["do"][1]), dev(lse), fscalar(448.0), fscalar(1024.0), dQ, dK, dV, workspace=ws)
        torch.cuda.synchronize()
        out.append((host_u16(dK), host_u16(dV)))
    assert np.all((out[1][0] & 0x7F80) != 0x7F80)
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


def bwd_dkdv(c, O, lse, do_bits, s, causal, rho_p, rho_ds):
    """dK and dV of one backward call with the scales given (the other outputs are covered elsewhere)."""
    B, H, S = lse.shape
    dQ, dK, dV = (torch.full((B, H, S, 128), 0x7FC0, dtype=torch.int16, device="cuda") for _ in range(3))
    ws = torch.empty(fog.fp8_attn_workspace(B, H, S, 128, True), dtype=torch.uint8, device="cuda")
    fog.fp8_attn_bwd(B, H, S, 128, s, causal, dev(c["q"][0]), dev(c["k"][0]), dev(c["v"][0]),
                     fscalar(c["q"][1]), fscalar(c["k"][1]), fscalar(c["v"][1]), dev(O), dev(do_bits), dev(c["do"][0]),
                     fscalar(c["do"][1]), dev(lse), fscalar(rho_p), fscalar(rho_ds), dQ, dK, dV, workspace=ws)
    torch.cuda.synchronize()
    return host_u16(dK), host_u16(dV)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("rho_p", [1000.0, 4096.0, 2.0 ** 40])
def test_backward_with_an_infinite_output_gradient_and_a_large_scale_of_p(rho_p, causal):
    """As above with a probability scale of 448 and beyond: rho_p P times the stand-in of an infinite D must not reach infinity
    in the casts.  dK and dV have to be those of a huge finite element, byte for byte."""
    B, H, S = 1, 2, 192
    q, k, v, do = synth.small_attention(2720, B, H, S)
    c = cast_all(q, k, v, do)
    s = 1 / math.sqrt(128)
    O, lse, _ = gpu_fwd(c, B, H, S, s, causal, want_amax=False)
    out = []
    for bits in (0x7F80, 0x7149):                  # +infinity, 1e30
        d = do.copy()
        d[0, 0, 100, 5] = bits
        out.append(bwd_dkdv(c, O, lse, d, s, causal, rho_p, 1024.0))
    assert np.all((out[0][0] & 0x7F80) != 0x7F80)
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("causal", [True, False])
def test_backward_dk_under_a_tiny_scale_of_p(causal):
    """dK does not depend on the scale of P but for rounding: under a scale of 2^-100 the row constant D rho_ds / rho_p is huge for
    ordinary gradients, and dK is that of scale 448 (which the oracle checks).  The two differ in the last bit of products taken
    in another order: codes of dS flip on rounding ties, at most one E5M2 step (an eighth to a quarter of the value) each."""
    B, H, S = 1, 2, 192
    q, k, v, do = synth.small_attention(2730, B, H, S)
    c = cast_all(q, k, v, do)
    s = 1 / math.sqrt(128)
    O, lse, _ = gpu_fwd(c, B, H, S, s, causal, want_amax=False)
    a, b = (synth.bf16_bits_to_f32(bwd_dkdv(c, O, lse, do, s, causal, rho_p, 2.0 ** 20)[0]).astype(np.float64) for rho_p in (448.0, 2.0 ** -100))
    assert np.isfinite(a).all() and np.abs(a).max() > 0
    assert np.linalg.norm(a - b) <= 5e-3 * np.linalg.norm(a)


@pytest.mark.parametrize("rho_ds", [1024.0, 2.0 ** 62])
def test_backward_keeps_a_nan_of_the_output_gradient(rho_ds):
    """A NaN in dO makes D of its row NaN: dK is NaN for every key that the row attends to, under a scale of dS that saturates
    everything else too, and for no other key."""
    B, H, S = 1, 2, 192
    q, k, v, do = synth.small_attention(2740, B, H, S)
    c = cast_all(q, k, v, do)
    s = 1 / math.sqrt(128)
    O, lse, _ = gpu_fwd(c, B, H, S, s, True, want_amax=False)
    d = do.copy()
    d[0, 1, 100, 5] = 0x7FC0
    dK, _ = bwd_dkdv(c, O, lse, d, s, True, 448.0, rho_ds)
    nan = (dK & 0x7FFF) > 0x7F80
    assert nan[0, 1, :101].all() and not nan[0, 1, 101:].any() and not nan[0, 0].any()


@pytest.mark.parametrize("name", ["q", "k", "v", "do"])
def test_backward_keeps_nan_codes_of_the_operands(name):
    """A NaN code in an operand reaches dK and dV wherever its row or column takes part, and no other head."""
    B, H, S = 1, 2, 192
    q, k, v, do = synth.small_attention(2750, B, H, S)
    c = cast_all(q, k, v, do)
    s = 1 / math.sqrt(128)
    c[name][0][0, 1, 100, 5] = 0x7F
    O, lse, _ = gpu_fwd(c, B, H, S, s, True, want_amax=False)
    dK, dV = ((x & 0x7FFF) > 0x7F80 for x in bwd_dkdv(c, O, lse, do, s, True, 448.0, 1024.0))
    assert not dK[0, 0].any() and not dV[0, 0].any()
    if name == "q":                    # scores of query 100
        assert dK[0, 1, :101].all() and dV[0, 1, :101].all()
    elif name == "k":                  # scores of key 100, and through lse every key of the queries from 100 on
        assert dK[0, 1].all() and dV[0, 1].all()
    elif name == "v":                  # dP of key 100, and through O (one column of it) D of the queries from 100 on
        assert dK[0, 1].all() and not dV[0, 1].any()
    else:                              # dP of query 100; dV in the element's own column
        assert dK[0, 1, :101].all()
        assert dV[0, 1, :101, 5].all() and not np.delete(dV[0, 1], 5, axis=1).any()


def gqa_case(seed, B, H, Hkv, S):
    """Grouped-query inputs: Q and dO with H heads, K and V with H_kv heads (same recipe, own seed)."""
    q, _, _, do = synth.small_attention(seed, B, H, S)
    _, k, v, _ = synth.small_attention(seed + 1, B, Hkv, S)
    return cast_all(q, k, v, do), do


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,H,Hkv,S", [(1, 2, 1, 128), (2, 4, 2, 320), (1, 8, 2, 192), (1, 4, 1, 448)])
def test_grouped_query_parity(B, H, Hkv, S, causal):
    """H_kv < H (Appendix B: grouped-query attention): forward per query head against its group's K/V,
    backward with dK/dV summed over the group."""
    c, do = gqa_case(3000 + S + H, B, H, Hkv, S)
    heads = [(b, h) for b in range(B) for h in range(H)]
    check_fwd(c, B, H, S, 1 / math.sqrt(128), causal, heads)
    run_bwd(c, B, H, S, 1 / math.sqrt(128), causal, heads, do)


@pytest.mark.parametrize("B,H,Hkv,S", [(2, 4, 2, 8192), (1, 2, 1, 16384)])
def test_long_context_grouped_query_sampled(B, H, Hkv, S):
    """Sequences of 8192 and 16384 tokens with grouped queries, causal, whole on the GPU; the oracle
    evaluates sampled outputs one by one.  Under the causal mask row i of O / lse / dQ depends on the
    keys 0..i only, and row j of dK / dV on the queries j..S-1 only, so each sample is the oracle's own
    (unmasked) routine on that slice of the head: no S x S matrix is ever formed.  The backward pass
    consumes the GPU's own forward results on both sides, as a training step does."""
    G = H // Hkv
    c, do = gqa_case(S + H, B, H, Hkv, S)
    s = 0.125
    O, lse, _ = gpu_fwd(c, B, H, S, s, True)
    assert np.isfinite(lse).all()
    rng = np.random.default_rng(S)
    rows = sorted({0, 1, 63, 64, 127, 128, S // 2 - 1, S // 2, S - 65, S - 64, S - 2, S - 1, *map(int, rng.integers(0, S, 6))})
    heads = [(0, 0), (B - 1, H - 1)]
    sq, sk, sv = c["q"][1], c["k"][1], c["v"][1]
    for (b, h) in heads:
        hk = h // G
        refs, slacks = [], []
        for i in rows:
            args = (c["q"][0][b, h, i:i + 1], c["k"][0][b, hk, :i + 1], c["v"][0][b, hk, :i + 1], sq, sk, sv)
            Or, lr, _ = attention.attn_fwd_head(*args, s, 448.0, False)
            dx = mfma_model.logit_uncertainty(args[0], args[1], sq, sk, s, False)
            refs.append(Or)
            slacks.append(mfma_model.fwd_cast_slack(*args, s, 448.0, False, dx=dx))
            lunc = mfma_model.lse_uncertainty(args[0], args[1], sq, sk, s, False, dx=dx)
            assert np.all(np.abs(lse[b, h, i:i + 1] - lr) <= 2e-4 + lunc)
        # the sampled rows of a head as one tensor; a third of them are short rows (0, 1, 63, 64, ...), where a
        # single two-code element of P moves the whole row
        check_attention(O[b, h, rows], np.concatenate(refs), np.concatenate(slacks), what="O[%d,%d] rows" % (b, h),
                        max_exceed_frac=SAMPLED_EXCEED)
    # backward on the GPU's own O and lse; the scale of dS from a first pass (delayed-style)
    Od, lsed = dev(O), dev(lse)
    dQ = torch.full((B, H, S, 128), 0x7FC0, dtype=torch.int16, device="cuda")
    dK, dV = (torch.full((B, Hkv, S, 128), 0x7FC0, dtype=torch.int16, device="cuda") for _ in range(2))
    am = torch.full((1,), -1.0, device="cuda")
    ws = torch.empty(fog.fp8_attn_workspace(B, H, S, 128, True, H_kv=Hkv), dtype=torch.uint8, device="cuda")
    dev_in = (dev(c["q"][0]), dev(c["k"][0]), dev(c["v"][0]), fscalar(sq), fscalar(sk), fscalar(sv), Od, dev(do), dev(c["do"][0]),
              fscalar(c["do"][1]), lsed, fscalar(448.0))
    fog.fp8_attn_bwd(B, H, S, 128, s, True, *dev_in, fscalar(1.0), dQ, dK, dV, amax_ds=am, workspace=ws, H_kv=Hkv)
    torch.cuda.synchronize()
    rho_ds, _ = scaling.compute_scale(np.float32(am.item()), fp8.E5M2)
    fog.fp8_attn_bwd(B, H, S, 128, s, True, *dev_in, fscalar(rho_ds), dQ, dK, dV, amax_ds=am, workspace=ws, H_kv=Hkv)
    torch.cuda.synchronize()
    dQ, dK, dV = host_u16(dQ), host_u16(dK), host_u16(dV)
    sdo = c["do"][1]

    def bwd_slice(b, h, qs, ks):
        """Oracle backward of query head (b, h) restricted to queries qs and keys ks (all visible)."""
        hk = h // G
        args = (c["q"][0][b, h, qs], c["k"][0][b, hk, ks], c["v"][0][b, hk, ks], sq, sk, sv,
                O[b, h, qs], do[b, h, qs], c["do"][0][b, h, qs], sdo, lse[b, h, qs], s, 448.0, rho_ds, False)
        return attention.attn_bwd_head(*args), mfma_model.bwd_cast_slack(*args)

    for (b, h) in heads:
        res = [bwd_slice(b, h, slice(i, i + 1), slice(0, i + 1)) for i in rows]
        check_attention(dQ[b, h, rows], np.concatenate([r[0] for r, _ in res]), np.concatenate([sl[0] for _, sl in res]),
                        what="dQ[%d,%d] rows" % (b, h), max_exceed_frac=SAMPLED_EXCEED)
    for (b, hk) in [(0, 0), (B - 1, Hkv - 1)]:
        dks, dvs, slks, slvs = [], [], [], []
        for j in rows:
            dk = dv = slk = slv = 0.0
            for h in range(hk * G, hk * G + G):            # the group's query heads all feed this key
                r, sl = bwd_slice(b, h, slice(j, S), slice(j, j + 1))
                dk, dv, slk, slv = dk + r[1], dv + r[2], slk + sl[1], slv + sl[2]
            dks.append(dk); dvs.append(dv); slks.append(slk); slvs.append(slv)
        check_attention(dK[b, hk, rows], np.concatenate(dks), np.concatenate(slks), what="dK[%d,%d] rows" % (b, hk),
                        max_exceed_frac=SAMPLED_EXCEED)
        check_attention(dV[b, hk, rows], np.concatenate(dvs), np.concatenate(slvs), what="dV[%d,%d] rows" % (b, hk),
                        max_exceed_frac=SAMPLED_EXCEED)


def test_backward_two_launch_form_noncausal():
    """Enough key blocks (B H_kv S / 128 >= 1024) for dK and dV to be produced by two launches instead of
    one; non-causal, two heads checked in full (config 3 below covers the causal case of that form)."""
    B, H, S = 8, 16, 1024
    q, k, v, do = synth.small_attention(4242, B, H, S)
    c = cast_all(q, k, v, do)
    run_bwd(c, B, H, S, 1 / math.sqrt(128), False, [(0, 0), (B - 1, H - 1)], do)


def test_config3_full_size_sampled_heads():
    """Config 3 whole on the GPU (B 4, H 16, S 2048, D 128, causal); the oracle checks 4 (batch, head)
    pairs in full (first, last, two seeded), forward and backward; every head is checked for sanity."""
    cfg = synth.CONFIGS[3]
    a = cfg.attn
    t = synth.attention_tensors(cfg)
    c = cast_all(t["Q"], t["K"], t["V"], t["dO"])
    rng = np.random.default_rng(3)
    heads = [(0, 0), (a.B - 1, a.H - 1)]
    while len(heads) < 4:
        bh = (int(rng.integers(a.B)), int(rng.integers(a.H)))
        if bh not in heads:
            heads.append(bh)
    s = 1 / math.sqrt(128)
    O, lse = check_fwd(c, a.B, a.H, a.S, s, True, heads)
    Of = bf16.bits_to_f64(O)
    assert np.isfinite(Of).all()
    # every output row is a convex combination of decoded V rows (up to the cast of P): bounded by max |V|
    vmax = np.abs(fp8.decode(c["v"][0], fp8.E4M3)).max() * float(c["v"][1])
    assert np.abs(Of).max() <= vmax * 1.07
    run_bwd(c, a.B, a.H, a.S, s, True, heads, t["dO"])


def test_optional_abs_max_outputs_may_be_null():
    """amax_p and amax_ds are optional: without them the kernels take the instantiations that skip the
    running maxima, and the results are bit-identical to the calls that report them."""
    B, H, S = 1, 2, 192
    q, k, v, do = synth.small_attention(909, B, H, S)
    c = cast_all(q, k, v, do)
    s = 0.125
    O1, lse1, _ = gpu_fwd(c, B, H, S, s, True, want_amax=True)
    O2, lse2, _ = gpu_fwd(c, B, H, S, s, True, want_amax=False)
    assert np.array_equal(O1, O2) and np.array_equal(lse1, lse2)
    res = []
    for with_amax in (True, False):
        dQ, dK, dV = (torch.full((B, H, S, 128), 0x7FC0, dtype=torch.int16, device="cuda") for _ in range(3))
        am = torch.zeros(1, device="cuda") if with_amax else None
        ws = torch.empty(fog.fp8_attn_workspace(B, H, S, 128, True), dtype=torch.uint8, device="cuda")
        fog.fp8_attn_bwd(B, H, S, 128, s, True, dev(c["q"][0]), dev(c["k"][0]), dev(c["v"][0]), fscalar(c["q"][1]), fscalar(c["k"][1]),
                         fscalar(c["v"][1]), dev(O1), dev(do), dev(c["do"][0]), fscalar(c["do"][1]), dev(lse1), fscalar(448.0),
                         fscalar(2.0 ** 20), dQ, dK, dV, amax_ds=am, workspace=ws)
        torch.cuda.synchronize()
        res.append([host_u16(x) for x in (dQ, dK, dV)])
    assert all(np.array_equal(a, b) for a, b in zip(*res))


def test_attention_argument_errors():
    lib = fog.load()
    st = torch.cuda.current_stream().cuda_stream
    x = torch.zeros(64 * 128, dtype=torch.uint8, device="cuda")
    o = torch.zeros(64 * 128, dtype=torch.int16, device="cuda")
    f = fscalar(1.0)
    l = torch.zeros(64, device="cuda")
    p, fp = x.data_ptr(), f.data_ptr()
    args = lambda D, S, q=p, H=1, Hkv=1: (1, H, Hkv, S, D, 0.1, 1, q, p, p, fp, fp, fp, fp, o.data_ptr(), l.data_ptr(), None, None, 0, st)
    assert lib.fog_fp8_attn_fwd(*args(64, 64)) == 4
    assert lib.fog_fp8_attn_fwd(*args(128, 48)) == 4
    assert lib.fog_fp8_attn_fwd(*args(128, 64, None)) == 1
    assert lib.fog_fp8_attn_fwd(*args(128, 64, p + 4)) == 3
    assert lib.fog_fp8_attn_fwd(*args(128, 64)) == 0
    assert lib.fog_fp8_attn_fwd(*args(128, 64, p, 3, 2)) == 2          # H not a multiple of H_kv
    assert lib.fog_fp8_attn_fwd(*args(128, 64, p, 2, 0)) == 2
    b = (1, 1, 1, 64, 128, 0.1, 1, p, p, p, fp, fp, fp, o.data_ptr(), o.data_ptr(), p, fp, l.data_ptr(), fp, fp,
         o.data_ptr(), o.data_ptr(), o.data_ptr(), None)
    assert lib.fog_fp8_attn_bwd(*b, None, 0, st) == 5
    ws = torch.zeros(3 * 64, device="cuda")
    assert lib.fog_fp8_attn_bwd(*b, ws.data_ptr(), 100, st) == 5
    assert lib.fog_fp8_attn_bwd(*b, ws.data_ptr(), 3 * 64 * 4, st) == 0
    torch.cuda.synchronize()


def test_forward_with_integer_logits_has_no_open_decision():
    """Inputs built so that every logit is a small integer in the log2 domain: every p is a power of two, whose
    E4M3 cast is the same whichever side evaluates it (powers of two sit far from rounding boundaries), so no
    slack is granted: O must meet the plain gate, lse a tight one.  Q~ rows are one-hot (1 or 2 at column
    i mod 128), K~ holds integers -3..3, both scales are 1 and s = ln 2, so x_ij = q_i k_j,(i mod 128)."""
    B, H, S = 1, 2, 320
    rng = np.random.default_rng(99)
    Q8 = np.zeros((B, H, S, 128), np.uint8)
    one, two = int(fp8.encode_sat(np.float32(1.0), fp8.E4M3)), int(fp8.encode_sat(np.float32(2.0), fp8.E4M3))
    for h in range(H):
        for i in range(S):
            Q8[0, h, i, i % 128] = one if rng.random() < 0.5 else two
    K8 = fp8.encode_sat(rng.integers(-3, 4, size=(B, H, S, 128)).astype(np.float32), fp8.E4M3)
    _, _, v, _ = synth.small_attention(98, B, H, S)
    rho_v, vinv = scaling.compute_scale(scaling.amax(v), fp8.E4M3)
    V8 = scaling.quantize(v.reshape(-1, 128), rho_v, fp8.E4M3).reshape(v.shape)
    c = {"q": (Q8, np.float32(1.0)), "k": (K8, np.float32(1.0)), "v": (V8, vinv)}
    s = float(np.float32(np.log(2.0)))
    for causal in (True, False):
        O, lse, am = gpu_fwd(c, B, H, S, s, causal)
        for h in range(H):
            x = attention.logits(Q8[0, h], K8[0, h], 1.0, 1.0, s, causal)
            fin = np.isfinite(x)
            assert np.abs(x[fin] - np.rint(x[fin])).max() < 1e-6 and np.ptp(x[fin]) >= 8      # integers, spread over many binades
            Or, lr, _ = attention.attn_fwd_head(Q8[0, h], K8[0, h], V8[0, h], 1.0, 1.0, vinv, s, 448.0, causal)
            st = check_bf16(O[0, h], Or, what="O, integer logits", max_flip_frac=0.1)
            assert st["max_steps"] <= 1
            assert np.abs(lse[0, h] - lr).max() < 2e-5


def test_backward_with_q_zero_closed_forms():
    """Q~ = 0: every logit is 0, P_ij = 1 / (i + 1) exactly and 448 / (i + 1) never comes near an E4M3 rounding
    boundary for i < 256, so the cast of P is decided alike on both sides: dV must meet the plain gate with no
    slack.  dK = s sinv_q / rho_ds (dS~^T Q~) is a sum of zeros: every element is exactly zero."""
    B, H, S = 1, 2, 256
    q, k, v, do = synth.small_attention(4321, B, H, S)
    c = cast_all(q, k, v, do)
    c["q"] = (np.zeros_like(c["q"][0]), np.float32(1.0))
    s = 0.125
    O_bits = np.zeros((B, H, S, 128), np.uint16)
    lse = np.zeros((B, H, S), np.float32)
    for h in range(H):
        Or, lr, _ = attention.attn_fwd_head(c["q"][0][0, h], c["k"][0][0, h], c["v"][0][0, h], c["q"][1], c["k"][1], c["v"][1], s, 448.0, True)
        O_bits[0, h] = bf16.f64_to_bits_rne(Or)
        lse[0, h] = lr.astype(np.float32)
        assert np.array_equal(lse[0, h], np.log2(np.arange(1, S + 1)).astype(np.float32))
    dQ, dK, dV = (torch.full((B, H, S, 128), 0x7FC0, dtype=torch.int16, device="cuda") for _ in range(3))
    ws = torch.empty(fog.fp8_attn_workspace(B, H, S, 128, True), dtype=torch.uint8, device="cuda")
    rho_ds = np.float32(2.0 ** 16)
    fog.fp8_attn_bwd(B, H, S, 128, s, True, dev(c["q"][0]), dev(c["k"][0]), dev(c["v"][0]), fscalar(c["q"][1]), fscalar(c["k"][1]),
                     fscalar(c["v"][1]), dev(O_bits), dev(do), dev(c["do"][0]), fscalar(c["do"][1]), dev(lse), fscalar(448.0),
                     fscalar(rho_ds), dQ, dK, dV, workspace=ws)
    torch.cuda.synchronize()
    dK, dV = host_u16(dK), host_u16(dV)
    assert np.all((dK & 0x7FFF) == 0)                      # exactly zero (either sign)
    for h in range(H):
        dov = fp8.decode(c["do"][0][0, h], fp8.E5M2) * np.float64(c["do"][1])
        pt = fp8.decode(fp8.encode_sat(np.float32(448.0 / np.arange(1, S + 1)), fp8.E4M3), fp8.E4M3) / 448.0
        want = np.stack([(pt[j:, None] * dov[j:]).sum(0) for j in range(S)])       # dV_j = sum_{i >= j} P~_ij dO_i
        r = attention.attn_bwd_head(c["q"][0][0, h], c["k"][0][0, h], c["v"][0][0, h], c["q"][1], c["k"][1], c["v"][1], O_bits[0, h],
                                    do[0, h], c["do"][0][0, h], c["do"][1], lse[0, h], s, 448.0, rho_ds, True)
        assert np.allclose(r[2], want, rtol=1e-12, atol=1e-18)
        check_bf16(dV[0, h], want, what="dV, Q = 0", max_flip_frac=0.1)


def test_failing_attention_calls_leave_device_memory_untouched():
    """Argument errors are detected before anything is launched: the optional abs-max outputs, which a
    successful call zeroes first, keep their contents when the call fails."""
    lib = fog.load()
    st = torch.cuda.current_stream().cuda_stream
    x = torch.zeros(64 * 128, dtype=torch.uint8, device="cuda")
    o = torch.full((64 * 128,), 0x1234, dtype=torch.int16, device="cuda")
    f = fscalar(1.0)
    l = torch.full((64,), -3.0, device="cuda")
    am = torch.full((1,), -7.0, device="cuda")
    p, fp = x.data_ptr(), f.data_ptr()
    fwd = lambda q, S=64, D=128: lib.fog_fp8_attn_fwd(1, 1, 1, S, D, 0.1, 1, q, p, p, fp, fp, fp, fp, o.data_ptr(), l.data_ptr(),
                                                       am.data_ptr(), None, 0, st)
    assert fwd(None) == 1 and fwd(p + 4) == 3 and fwd(p, S=48) == 4 and fwd(p, D=64) == 4
    bwd = lambda q, ws, wsb: lib.fog_fp8_attn_bwd(1, 1, 1, 64, 128, 0.1, 1, q, p, p, fp, fp, fp, o.data_ptr(), o.data_ptr(), p, fp,
                                                  l.data_ptr(), fp, fp, o.data_ptr(), o.data_ptr(), o.data_ptr(), am.data_ptr(), ws, wsb, st)
    ws = torch.zeros(3 * 64, device="cuda")
    assert bwd(None, ws.data_ptr(), 3 * 64 * 4) == 1 and bwd(p + 4, ws.data_ptr(), 3 * 64 * 4) == 3 and bwd(p, None, 0) == 5
    assert bwd(p, ws.data_ptr(), 100) == 5
    torch.cuda.synchronize()
    assert am.item() == -7.0 and (o == 0x1234).all() and (l == -3.0).all() and (ws == 0).all()
    assert fwd(p) == 0                                   # the same arguments, valid: the call runs and zeroes the abs-max first
    torch.cuda.synchronize()
    assert am.item() != -7.0


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,H,Hkv,S", [(3, 45, 45, 64), (2, 33, 33, 128), (1, 6, 2, 64), (1, 3, 1, 192)])
def test_backward_workgroup_shapes(B, H, Hkv, S, causal):
    """dK/dV with 64 keys per workgroup (more than 128 of them) and with 32 keys and two pairs that take the query blocks in
    turns (few workgroups; an odd number of blocks leaves one turn empty): first, last and middle heads against the oracle."""
    c, do = gqa_case(3400 + S + H, B, H, Hkv, S)
    G = H // Hkv
    heads = sorted({(b, h) for b in (0, B - 1) for hk in (0, Hkv // 2, Hkv - 1) for h in range(hk * G, hk * G + G)})
    run_bwd(c, B, H, S, 1 / math.sqrt(128), causal, heads, do)


@pytest.mark.parametrize("B,H,Hkv,S", [(1, 1, 1, 64), (2, 3, 3, 192), (1, 8, 1, 320), (1, 72, 1, 64)])
def test_backward_abs_max_sees_every_row(B, H, Hkv, S):
    """max |dS| wherever its row lies: the dQ kernel leaves one maximum per 32 rows, workgroups of the dK/dV kernel reduce shares of
    them.  Only one row has an output gradient, so every other row contributes 0.  With the smaller workspace dK and dV are summed in one
    piece, by fewer workgroups: the last case has two then, whose shares of 72 maxima are more than a wave holds, and rows among the last
    eight of both."""
    g = torch.Generator().manual_seed(H * S)
    codes = lambda rows: torch.randint(0x28, 0x40, (rows, 128), generator=g, dtype=torch.uint8) | (torch.randint(0, 2, (rows, 128), generator=g, dtype=torch.uint8) << 7)
    q, k, v = (codes(B * h * S).cuda() for h in (H, Hkv, Hkv))
    f64 = lambda t: t.view(torch.float8_e4m3fn).double()
    one, s = fscalar(1.0), 0.05
    O = torch.empty((B * H * S, 128), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty(B * H * S, device="cuda")
    fog.fp8_attn_fwd(B, H, S, 128, s, False, q, k, v, one, one, one, fscalar(448.0), O, lse, H_kv=Hkv)
    dQ, dK, dV = (torch.empty((B * h * S, 128), dtype=torch.bfloat16, device="cuda") for h in (H, Hkv, Hkv))
    ws = torch.empty(fog.fp8_attn_workspace(B, H, S, 128, True, H_kv=Hkv), dtype=torch.uint8, device="cuda")
    groups = B * H * S // 32
    rows_only = ws[:3 * B * H * S * 4]
    for n in range(0, groups, max(1, groups // 24)):
        row = 32 * n + (7 * n + 3) % 32
        do = torch.zeros((B * H * S, 128), dtype=torch.bfloat16, device="cuda")
        do[row] = (torch.arange(128, device="cuda") % 7 - 3).to(torch.bfloat16)      # values that E5M2 holds exactly
        am = torch.full((2,), 9.0, device="cuda")
        for i, room in enumerate((ws, rows_only)):
            fog.fp8_attn_bwd(B, H, S, 128, s, False, q, k, v, one, one, one, O, do, do.to(torch.float8_e5m2).view(torch.uint8), one, lse,
                             fscalar(448.0), one, dQ, dK, dV, amax_ds=am[i:], workspace=room, H_kv=Hkv)
        kv = row // S // (H // Hkv) * S
        kk, vv, d = f64(k[kv:kv + S]), f64(v[kv:kv + S]), do[row].double()
        p = torch.softmax(s * (kk @ f64(q[row])), dim=0)
        want = (p * (vv @ d - (d * O[row].double()).sum())).abs().max().item()
        assert abs(am[0].item() - want) <= 1e-4 * want      # binary32 sums of 128 terms and one exponential: 1e-5 at most
        assert am[1].item() == am[0].item()


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,H,Hkv,S", [(1, 4, 1, 512), (1, 4, 1, 768), (1, 34, 2, 128), (1, 16, 1, 192), (1, 130, 1, 64)])
def test_backward_in_parts(B, H, Hkv, S, causal):
    """Few keys and long streams of query blocks: dK and dV summed in two, three, two, three and eight parts (parts that end inside a
    head, odd numbers of blocks, streams of late keys that are shorter than the parts are many), against the oracle and against the
    sums in one piece."""
    rows = 3 * B * H * S * 4
    assert fog.fp8_attn_workspace(B, H, S, 128, True, H_kv=Hkv) > rows
    c, do = gqa_case(3900 + S + H, B, H, Hkv, S)
    s = 1 / math.sqrt(128)
    if H // Hkv <= 4:   # the slacks of a group's casts add up: without a mask, those of 8 heads exceed what the oracle's check allows a group
        run_bwd(c, B, H, S, s, causal, [(b, h) for b in range(B) for h in range(H // Hkv)], do)
    # the smaller workspace and one that is not 16-byte aligned keep working; the sums then differ in the order of binary32 additions
    O, lse, _ = gpu_fwd(c, B, H, S, s, causal, want_amax=False)
    args = (dev(c["q"][0]), dev(c["k"][0]), dev(c["v"][0]), fscalar(c["q"][1]), fscalar(c["k"][1]), fscalar(c["v"][1]), dev(O), dev(do),
            dev(c["do"][0]), fscalar(c["do"][1]), dev(lse), fscalar(448.0), fscalar(64.0))
    full = torch.empty(fog.fp8_attn_workspace(B, H, S, 128, True, H_kv=Hkv) + 16, dtype=torch.uint8, device="cuda")
    out = []
    for ws in (full, full[:rows], full[4:]):
        o = [torch.full((B, h, S, 128), float("nan"), dtype=torch.bfloat16, device="cuda") for h in (H, Hkv, Hkv)] + [torch.zeros(1, device="cuda")]
        fog.fp8_attn_bwd(B, H, S, 128, s, causal, *args, *o[:3], amax_ds=o[3], workspace=ws, H_kv=Hkv)
        torch.cuda.synchronize()
        out.append(o)
    for o in out[1:]:
        assert torch.equal(o[0], out[0][0]) and torch.equal(o[3], out[0][3])
        for a, b in zip(o[1:3], out[0][1:3]):
            # one bf16 step where the sums straddle a rounding boundary, and binary32 sums of up to 8320 terms where they cancel
            a, b = a.double(), b.double()
            assert ((a - b).abs() <= 2.0 ** -7 * b.abs() + 1e-5 * b.abs().max()).all()
    assert torch.equal(out[1][1], out[2][1]) and torch.equal(out[1][2], out[2][2])


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("S", [320, 576, 704])
@pytest.mark.parametrize("steps", [(1, 2, 3, 5, 6), (0, 14, 16, 30, 32), (0, 16, 18, 64, 72), (0, 32, 128, 256, 448), (448, 128, 32, 1, 0)])
def test_forward_with_growing_row_references(steps, S, causal):
    """O stays relative to an earlier row reference until the reference has grown by more than 32.  Integer logits (as above) that grow from key
    block to key block: by little, to 32 and 64 (rows of q = 1 and 2 share a wave, so one moves O and the other has to follow), by more than
    32 at every block, and not at all.  S = 320 takes a block in one go, the longer ones its scores a block ahead and P V a block behind: there the
    first has the bytes it has among many copies.  A V of 2^-93 times the size gives exactly 2^-93 times the O: nothing on the way
    leaves binary32's range."""
    H = 2
    rng = np.random.default_rng(sum(steps))
    Q8 = np.zeros((1, H, S, 128), np.uint8)
    one, two = int(fp8.encode_sat(np.float32(1.0), fp8.E4M3)), int(fp8.encode_sat(np.float32(2.0), fp8.E4M3))
    for h in range(H):
        for i in range(S):
            Q8[0, h, i, i % 128] = one if rng.random() < 0.5 else two
    of_block = np.rint(np.interp(np.linspace(0, 4, S // 64), np.arange(5), steps)).astype(np.float32)
    k = np.repeat(of_block, 64)[None, None, :, None] - rng.integers(0, 3, size=(1, H, S, 128)).astype(np.float32)
    K8 = fp8.encode_sat(k, fp8.E4M3)                       # integers on the E4M3 grid
    _, _, v, _ = synth.small_attention(97, 1, H, S)
    rho_v, vinv = scaling.compute_scale(scaling.amax(v), fp8.E4M3)
    V8 = scaling.quantize(v.reshape(-1, 128), rho_v, fp8.E4M3).reshape(v.shape)
    c = {"q": (Q8, np.float32(1.0)), "k": (K8, np.float32(1.0)), "v": (V8, vinv)}
    s = float(np.float32(np.log(2.0)))
    O, lse, am = gpu_fwd(c, 1, H, S, s, causal)
    for h in range(H):
        Or, lr, _ = attention.attn_fwd_head(Q8[0, h], K8[0, h], V8[0, h], 1.0, 1.0, vinv, s, 448.0, causal)
        check_bf16(O[0, h], Or, what="O, growing references", max_flip_frac=0.1)
        # s is ln 2 in binary32 (2^-25 relative) and so is its product with log2 e: at 896 the logits are 1e-4 off integers
        assert np.all(np.abs(lse[0, h] - lr) <= 2e-5 + 2.0 ** -22 * np.abs(lr))
    Os, lses, _ = gpu_fwd({**c, "v": (V8, np.ldexp(vinv, -93))}, 1, H, S, s, causal)
    assert np.array_equal(bf16.bits_to_f64(Os), np.ldexp(bf16.bits_to_f64(O), -93)) and np.array_equal(lses, lse)
    if S > 320:
        many = {n: (np.tile(x, (1, 150, 1, 1)), inv) for n, (x, inv) in c.items()}
        Om, lm, am_many = gpu_fwd(many, 1, 150 * H, S, s, causal)
        assert np.array_equal(Om, np.tile(O, (1, 150, 1, 1))) and np.array_equal(lm, np.tile(lse, (1, 150, 1))) and am_many == am


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("S", [512, 576, 640, 704, 1088])
def test_forward_of_few_workgroups_equals_that_of_many(S, causal):
    """Launches of few workgroups produce scores a block ahead, larger ones do not: the same operations in the same order, so one head
    by itself has the bytes it has among 300 copies (S = 512 is the shortest of the first kind; 8, 9, 10, 11 and 17 blocks: the walk over four stages ends in each)."""
    g = torch.Generator(device="cuda").manual_seed(S)
    q, k, v = ((torch.randn((1, S, 128), device="cuda", generator=g) * 64).to(torch.float8_e4m3fn).view(torch.uint8) for _ in range(3))
    inv, out = fscalar(2.0 ** -6), []
    for H in (1, 300):
        O, lse, am = torch.empty((H, S, 128), dtype=torch.bfloat16, device="cuda"), torch.empty((H, S), device="cuda"), fscalar(-1.0)
        rep = [x.expand(H, S, 128).contiguous() for x in (q, k, v)]
        fog.fp8_attn_fwd(1, H, S, 128, 1 / math.sqrt(128), causal, *rep, inv, inv, inv, fscalar(448.0), O, lse, amax_p=am)
        out.append((O, lse, am))
    assert torch.isfinite(out[0][0]).all() and out[0][0].abs().max() > 0
    assert (out[1][0] == out[0][0]).all() and (out[1][1] == out[0][1]).all() and torch.equal(out[1][2], out[0][2])
