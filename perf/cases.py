"""Performance cases of the FP8 hot path: what a training or inference program built on this library has it do.

Four kinds of case:
  linear    one linear layer of a training step: casts of X, W (E4M3) and dY (E5M2), then the forward, data-gradient and
            weight-gradient products (or the forward alone), under just-in-time or delayed scaling
  attention one attention layer: casts of Q, K, V (and dO), forward, and the backward where a training step has it
  producer  one element-wise producer of FP8 operands over a layer's activations
  ffn       the feed-forward half of a block as one forward pass: casts, up projection, GeLU + cast, down projection,
            post-norm + residual + cast

Everything goes through the ctypes binding paper_2505_20524_amd.fog; torch holds the device buffers.
"""
import math

import torch

from paper_2505_20524_amd import fog

E4M3, E5M2 = fog.E4M3, fog.E5M2
FP8_MAX = {E4M3: 448.0, E5M2: 57344.0}
FP8_DTYPE = {E4M3: torch.float8_e4m3fn, E5M2: torch.float8_e5m2}
HEAD_DIM = 128
HISTORY = 1024          # length of the abs-max history under delayed scaling
DO_STD = 1e-2           # output gradient of an attention layer
DY_STD = 1e-3           # output gradient of a linear layer
SCALE_DS = 65536.0      # what an earlier step's abs-max of dS would give for such gradients
GAIN = 1.0
ALPHA_P, ALPHA_N, ALPHA_T = 0.8, 0.8, 0.5

# the costliest listed cases bound the drawn ones
MAX_LINEAR = 8192 * 4096 * 14336
MAX_ATTENTION = 2 * 32 * 4096 * 4096
MAX_ELEMENTS = 8192 * 14336


def listed():
    return [
        # the smallest layer anyone runs: a projection of 512 tokens, forward only, where launches and latency count
        {"name": "linear fwd 512x1024x1024", "kind": "linear", "M": 512, "N": 1024, "K": 1024, "backward": False, "scaling": "jit"},
        # a batch whose token count and feature sizes fit no tile
        {"name": "linear ragged 1777x3088x2064", "kind": "linear", "M": 1777, "N": 3088, "K": 2064, "backward": True, "scaling": "jit"},
        # an ordinary layer, with transposed copies from the cast for the weight gradient
        {"name": "linear 4096x8192x2048 transposed", "kind": "linear", "M": 4096, "N": 8192, "K": 2048, "backward": True, "scaling": "jit_transposed"},
        # the largest layer of an 8B-scale block (its down projection) under delayed scaling
        {"name": "linear 8192x4096x14336 delayed", "kind": "linear", "M": 8192, "N": 4096, "K": 14336, "backward": True, "scaling": "delayed"},
        # a short ragged sequence with grouped queries: a fine-tuning batch of one
        {"name": "attention train 1x16/4x576", "kind": "attention", "B": 1, "H": 16, "H_kv": 4, "S": 576, "causal": True, "backward": True, "producer": "jit"},
        # attention of a 1.5B-scale block
        {"name": "attention train 4x16x2048", "kind": "attention", "B": 4, "H": 16, "H_kv": 16, "S": 2048, "causal": True, "backward": True, "producer": "jit"},
        # attention of an 8B-scale block
        {"name": "attention train 2x32x4096", "kind": "attention", "B": 2, "H": 32, "H_kv": 32, "S": 4096, "causal": True, "backward": True, "producer": "jit"},
        # long-context forward with grouped queries, Q and K from the fused normalisation
        {"name": "attention fwd 1x32/8x8192", "kind": "attention", "B": 1, "H": 32, "H_kv": 8, "S": 8192, "causal": True, "backward": False, "producer": "rmsnorm"},
        # the QK normalisation of an 8B-scale block: every head vector of 8192 tokens
        {"name": "qk rmsnorm 262144x128", "kind": "producer", "op": "rmsnorm", "rows": 262144, "cols": 128},
        # the feed-forward activation of an 8B-scale block
        {"name": "xielu 8192x14336", "kind": "producer", "op": "xielu", "rows": 8192, "cols": 14336},
        # the residual update of an 8B-scale block
        {"name": "postnorm 8192x4096", "kind": "producer", "op": "postnorm", "rows": 8192, "cols": 4096},
        # a whole feed-forward half of a 1.5B-scale block, forward
        {"name": "ffn 4096x2048x8192", "kind": "ffn", "T": 4096, "hidden": 2048, "inner": 8192},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "attention", "attention", "attention", "producer", "producer", "ffn"])
    if kind == "linear":
        while True:
            M, N, K = round(_log(rng, 64, 16384)), 16 * round(_log(rng, 256, 14336) / 16), 16 * round(_log(rng, 256, 14336) / 16)
            if 64 * 256 * 256 <= M * N * K <= MAX_LINEAR:
                break
        scaling = rng.choice(["jit", "jit", "delayed", "jit_transposed"])
        if scaling == "jit_transposed":
            M = max(16, M // 16 * 16)       # the transposed operands are contracted over the tokens
        return {"kind": kind, "M": M, "N": N, "K": K, "backward": scaling == "jit_transposed" or rng.random() < 0.75, "scaling": scaling}
    if kind == "attention":
        while True:
            B, H_kv, G = rng.randint(1, 4), rng.choice([1, 2, 4, 8, 16]), rng.choice([1, 1, 2, 4])
            S = 64 * round(_log(rng, 128, 8192) / 64)
            if B * H_kv * G * S * S <= MAX_ATTENTION:
                break
        return {"kind": kind, "B": B, "H": H_kv * G, "H_kv": H_kv, "S": S, "causal": rng.random() < 0.8, "backward": rng.random() < 0.7,
                "producer": rng.choice(["jit", "rmsnorm", "tanh"])}
    if kind == "producer":
        op = rng.choice(["rmsnorm", "tanh", "xielu", "gelu", "postnorm"])
        if op in ("rmsnorm", "tanh"):
            return {"kind": kind, "op": op, "rows": round(_log(rng, 1024, MAX_ELEMENTS // HEAD_DIM)), "cols": HEAD_DIM}
        while True:
            rows, cols = round(_log(rng, 256, 16384)), round(_log(rng, 512, 14336 if op != "postnorm" else 8192))
            if op == "postnorm":
                cols = 512 * max(1, round(cols / 512)) if rng.random() < 0.8 else 8 * round(cols / 8)
            else:
                cols = 16 * round(cols / 16) if rng.random() < 0.8 else cols
            if rows * cols <= MAX_ELEMENTS // (2 if op == "postnorm" else 1):
                break
        return {"kind": kind, "op": op, "rows": rows, "cols": cols}
    while True:
        T, hidden, inner = round(_log(rng, 128, 8192)), 64 * round(_log(rng, 512, 4096) / 64), 64 * round(_log(rng, 1024, 14336) / 64)
        if T * hidden * inner <= MAX_LINEAR // 2:
            return {"kind": kind, "T": T, "hidden": hidden, "inner": inner}


# ---------------------------------------------------------------------------------------------- inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, shape, std=1.0):
    return torch.randn(shape, device="cuda", generator=g).mul_(std).to(torch.bfloat16)


def _activations(g, rows, cols):
    """Normal values with two channels fifty times larger: the outliers of trained activations."""
    x = torch.randn((rows, cols), device="cuda", generator=g)
    at = torch.randperm(cols, device="cuda", generator=g)[:2]
    x[:, at] *= 50.0
    return x.to(torch.bfloat16)


def _float(value=0.0):
    return torch.full((1,), value, device="cuda")


def _bytes(n):
    return torch.empty(max(int(n), 16), dtype=torch.uint8, device="cuda")


def _bf16(*shape):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda")


class _Cast:
    """A bf16 tensor and where its FP8 cast goes."""

    def __init__(self, x, fmt, transposed=False):
        self.x, self.fmt = x, fmt
        self.q = torch.empty(x.shape, dtype=torch.uint8, device="cuda")
        self.qT = torch.empty((x.shape[1], x.shape[0]), dtype=torch.uint8, device="cuda") if transposed else None
        self.amax, self.scale, self.sinv = _float(), _float(1.0), _float(1.0)


class _Casts:
    """The casts of a layer's tensors: one batched call, or one call each where a transposed copy is wanted."""

    def __init__(self, casts, scaling):
        self.scaling = scaling
        self.single = [c for c in casts if c.qT is not None]
        self.batch = [c for c in casts if c.qT is None]
        if scaling == "delayed":
            for c in self.batch:
                # what the earlier steps left: abs-maxes a little above this step's
                c.history = torch.full((HISTORY,), 1.05, device="cuda") * c.x.abs().max().float()
                c.state = torch.zeros(fog.quantize_delayed_state(), dtype=torch.uint8, device="cuda")
            self.jobs = fog.make_delayed_jobs([(c.x, c.fmt, c.q, c.history, c.state, c.amax, c.scale, c.sinv) for c in self.batch])
            self.step = 0
        else:
            self.jobs = fog.make_cast_jobs([(c.x, c.fmt, c.q, c.amax, c.scale, c.sinv) for c in self.batch])
            self.ws = _bytes(fog.quantize_jit_batch_workspace(len(self.batch)))
            self.ws_single = _bytes(fog.quantize_jit_workspace())

    def run(self):
        if self.scaling == "delayed":
            fog.quantize_delayed_batch(self.jobs, self.step)
            self.step += 1
            return
        if self.batch:
            fog.quantize_jit_batch(self.jobs, self.ws)
        for c in self.single:
            fog.quantize_jit(c.x, c.fmt, c.amax, c.scale, c.sinv, self.ws_single, q=c.q, qT=c.qT)


def _gemm_workspace(*shapes):
    need = max(fog.fp8_gemm_workspace(*s) for s in shapes)
    return torch.empty(need, dtype=torch.uint8, device="cuda") if need else None


def _prepare_linear(case, g):
    M, N, K = case["M"], case["N"], case["K"]
    tr = case["scaling"] == "jit_transposed"
    st = {"case": case, "X": _Cast(_activations(g, M, K), E4M3, tr), "W": _Cast(_normal(g, (N, K), 0.02), E4M3), "Y": _bf16(M, N)}
    casts, shapes = [st["X"], st["W"]], [(fog.NT, M, N, K)]
    if case["backward"]:
        st["dY"] = _Cast(_normal(g, (M, N), DY_STD), E5M2, tr)
        st["dX"], st["dW"] = _bf16(M, K), _bf16(N, K)
        casts.append(st["dY"])
        shapes += [(fog.NN, M, K, N), (fog.NT if tr else fog.TN, N, K, M)]
    st["casts"] = _Casts(casts, case["scaling"])
    st["ws"] = _gemm_workspace(*shapes)
    return st


def _run_linear(st):
    case, X, W = st["case"], st["X"], st["W"]
    M, N, K, ws = case["M"], case["N"], case["K"], st["ws"]
    st["casts"].run()
    fog.fp8_gemm(fog.NT, M, N, K, X.q, E4M3, X.sinv, W.q, E4M3, W.sinv, st["Y"], workspace=ws)
    out = {"Y": st["Y"], "Xq": X.q, "Wq": W.q, "sX": X.scale, "sW": W.scale}
    if case["backward"]:
        dY = st["dY"]
        fog.fp8_gemm(fog.NN, M, K, N, dY.q, E5M2, dY.sinv, W.q, E4M3, W.sinv, st["dX"], workspace=ws)
        if dY.qT is not None:
            fog.fp8_gemm(fog.NT, N, K, M, dY.qT, E5M2, dY.sinv, X.qT, E4M3, X.sinv, st["dW"], workspace=ws)
            out.update(XqT=X.qT, dYqT=dY.qT)
        else:
            fog.fp8_gemm(fog.TN, N, K, M, dY.q, E5M2, dY.sinv, X.q, E4M3, X.sinv, st["dW"], workspace=ws)
        out.update(dX=st["dX"], dW=st["dW"], dYq=dY.q, sdY=dY.scale)
    return out


def _prepare_attention(case, g):
    B, H, Hk, S = case["B"], case["H"], case["H_kv"], case["S"]
    st = {"case": case, "s": 1.0 / math.sqrt(HEAD_DIM)}
    for name, heads in (("Q", H), ("K", Hk), ("V", Hk)):
        st[name] = _Cast(_normal(g, (B * heads * S, HEAD_DIM)), E4M3)
    st["O"], st["lse"] = _bf16(B * H * S, HEAD_DIM), torch.empty(B * H * S, device="cuda")
    st["scale_p"], st["scale_ds"], st["amax_p"], st["amax_ds"] = _float(448.0), _float(SCALE_DS), _float(), _float()
    casts = [st["V"]]
    if case["producer"] == "jit":
        casts = [st["Q"], st["K"], st["V"]]
    else:
        # a constant scale that cannot saturate: |y| <= sqrt(128) after the normalisation, 1 after tanh
        rho = 448.0 / (GAIN * math.sqrt(HEAD_DIM)) if case["producer"] == "rmsnorm" else 448.0
        for name in ("Q", "K"):
            st[name].scale.fill_(rho)
            st[name].sinv.copy_(1.0 / st[name].scale)
    if case["backward"]:
        st["dO"] = _Cast(_normal(g, (B * H * S, HEAD_DIM), DO_STD), E5M2)
        casts.append(st["dO"])
        st["dQ"], st["dK"], st["dV"] = _bf16(B * H * S, HEAD_DIM), _bf16(B * Hk * S, HEAD_DIM), _bf16(B * Hk * S, HEAD_DIM)
        st["ws"] = _bytes(fog.fp8_attn_workspace(B, H, S, HEAD_DIM, True, H_kv=Hk))
    st["casts"] = _Casts(casts, "jit")
    return st


def _run_attention(st):
    case, Q, K, V = st["case"], st["Q"], st["K"], st["V"]
    B, H, Hk, S, causal = case["B"], case["H"], case["H_kv"], case["S"], case["causal"]
    st["casts"].run()
    if case["producer"] != "jit":
        for c in (Q, K):
            if case["producer"] == "rmsnorm":
                fog.rmsnorm_quantize(c.x, E4M3, c.scale, c.q, gain=GAIN, amax_out=c.amax)
            else:
                fog.tanh_quantize(c.x, ALPHA_T, E4M3, c.scale, c.q)
    fog.fp8_attn_fwd(B, H, S, HEAD_DIM, st["s"], causal, Q.q, K.q, V.q, Q.sinv, K.sinv, V.sinv, st["scale_p"], st["O"], st["lse"],
                     amax_p=st["amax_p"], H_kv=Hk)
    out = {"O": st["O"], "lse": st["lse"], "amax_p": st["amax_p"]}
    if case["backward"]:
        dO = st["dO"]
        fog.fp8_attn_bwd(B, H, S, HEAD_DIM, st["s"], causal, Q.q, K.q, V.q, Q.sinv, K.sinv, V.sinv, st["O"], dO.x, dO.q, dO.sinv, st["lse"],
                         st["scale_p"], st["scale_ds"], st["dQ"], st["dK"], st["dV"], amax_ds=st["amax_ds"], workspace=st["ws"], H_kv=Hk)
        out.update(dQ=st["dQ"], dK=st["dK"], dV=st["dV"], amax_ds=st["amax_ds"])
    return out


def _producer_scale(op):
    """The scale a history of such activations gives (constant here, with some room above)."""
    return {"rmsnorm": 448.0 / math.sqrt(HEAD_DIM), "tanh": 448.0, "xielu": 448.0 / 36.0, "gelu": 448.0 / 6.5, "postnorm": 448.0 / 260.0}[op]


def _prepare_producer(case, g):
    rows, cols, op = case["rows"], case["cols"], case["op"]
    st = {"case": case, "x": _activations(g, rows, cols) if op == "postnorm" else _normal(g, (rows, cols)),
          "scale": _float(_producer_scale(op)), "amax": _float(), "q": torch.empty((rows, cols), dtype=torch.uint8, device="cuda")}
    if op == "postnorm":
        st["y"], st["xnew"] = _activations(g, rows, cols), _bf16(rows, cols)
        st["gamma"] = torch.randn(cols, device="cuda", generator=g) * 0.05 + 1.0 / math.sqrt(32.0)
    return st


def _run_producer(st):
    op, x, q, sc, am = st["case"]["op"], st["x"], st["q"], st["scale"], st["amax"]
    if op == "rmsnorm":
        fog.rmsnorm_quantize(x, E4M3, sc, q, gain=GAIN, amax_out=am)
    elif op == "tanh":
        fog.tanh_quantize(x, ALPHA_T, E4M3, sc, q, amax_out=am)
    elif op == "xielu":
        fog.xielu_quantize(x, ALPHA_P, ALPHA_N, E4M3, sc, q, amax_out=am)
    elif op == "gelu":
        fog.gelu_quantize(x, E4M3, sc, q, amax_out=am)
    else:
        fog.postnorm_residual_quantize(x, st["y"], st["gamma"], E4M3, sc, st["xnew"], q=q, amax_out=am)
        return {"xnew": st["xnew"], "q": q.view(torch.float8_e4m3fn), "amax": am}
    return {"q": q.view(torch.float8_e4m3fn), "amax": am}


def _prepare_ffn(case, g):
    T, D, F = case["T"], case["hidden"], case["inner"]
    st = {"case": case, "X": _Cast(_activations(g, T, D), E4M3), "W1": _Cast(_normal(g, (F, D), 0.02), E4M3), "W2": _Cast(_normal(g, (D, F), 0.02), E4M3)}
    st["casts"] = _Casts([st["X"], st["W1"], st["W2"]], "jit")
    st["h"], st["y"], st["xnew"] = _bf16(T, F), _bf16(T, D), _bf16(T, D)
    st["hq"], st["xq"] = torch.empty((T, F), dtype=torch.uint8, device="cuda"), torch.empty((T, D), dtype=torch.uint8, device="cuda")
    st["gamma"] = torch.randn(D, device="cuda", generator=g) * 0.05 + 1.0 / math.sqrt(32.0)
    st["scale_h"], st["scale_x"], st["amax_h"], st["amax_x"] = _float(448.0 / 40.0), _float(448.0 / 260.0), _float(), _float()
    st["sinv_h"] = 1.0 / st["scale_h"]
    st["ws"] = _gemm_workspace((fog.NT, T, F, D), (fog.NT, T, D, F))
    return st


def _run_ffn(st):
    case, X, W1, W2, ws = st["case"], st["X"], st["W1"], st["W2"], st["ws"]
    T, D, F = case["T"], case["hidden"], case["inner"]
    st["casts"].run()
    fog.fp8_gemm(fog.NT, T, F, D, X.q, E4M3, X.sinv, W1.q, E4M3, W1.sinv, st["h"], workspace=ws)
    fog.gelu_quantize(st["h"], E4M3, st["scale_h"], st["hq"], amax_out=st["amax_h"])
    fog.fp8_gemm(fog.NT, T, D, F, st["hq"], E4M3, st["sinv_h"], W2.q, E4M3, W2.sinv, st["y"], workspace=ws)
    fog.postnorm_residual_quantize(X.x, st["y"], st["gamma"], E4M3, st["scale_x"], st["xnew"], q=st["xq"], amax_out=st["amax_x"])
    return {"h": st["h"], "hq": st["hq"].view(torch.float8_e4m3fn), "y": st["y"], "xnew": st["xnew"],
            "xq": st["xq"].view(torch.float8_e4m3fn), "amax_h": st["amax_h"], "amax_x": st["amax_x"]}


_PREPARE = {"linear": _prepare_linear, "attention": _prepare_attention, "producer": _prepare_producer, "ffn": _prepare_ffn}
_RUN = {"linear": _run_linear, "attention": _run_attention, "producer": _run_producer, "ffn": _run_ffn}


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, _generator(seed))


def run(state):
    return _RUN[state["case"]["kind"]](state)


# ---------------------------------------------------------------------------------------------- work, tolerance
def work(case):
    if case["kind"] == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        n_in = M * K + N * K + (M * N if case["backward"] else 0)
        n_out = M * N + (M * K + N * K if case["backward"] else 0)
        copies = M * K + M * N if case["scaling"] == "jit_transposed" else 0
        return {"bytes": 3 * n_in + copies + 2 * n_out, "flops": 2 * M * N * K * (3 if case["backward"] else 1)}
    if case["kind"] == "attention":
        q, kv = case["B"] * case["H"] * case["S"] * HEAD_DIM, case["B"] * case["H_kv"] * case["S"] * HEAD_DIM
        fwd = 4 * case["B"] * case["H"] * case["S"] ** 2 * HEAD_DIM // (2 if case["causal"] else 1)
        # Q, K, V read and cast, O written; the backward also reads and casts dO and writes three gradients
        nbytes = 3 * (q + 2 * kv) + 2 * q + (3 * q + 2 * (q + 2 * kv) if case["backward"] else 0)
        return {"bytes": nbytes, "flops": fwd * 7 // 2 if case["backward"] else fwd}
    if case["kind"] == "producer":
        return {"bytes": (7 if case["op"] == "postnorm" else 3) * case["rows"] * case["cols"], "flops": 0}
    T, D, F = case["T"], case["hidden"], case["inner"]
    return {"bytes": 3 * (T * D + 2 * D * F) + 3 * T * F + 3 * T * D, "flops": 4 * T * D * F}


def tolerance(case):
    if case["kind"] == "linear":
        # casts to the byte; products summed in 32 bits in another order, one rounding to bf16 (unit roundoff 2^-9)
        return {"rel": 2e-3, "max": 0.02, "differ": 0.0}
    if case["kind"] == "attention":
        # a probability or dS next to a rounding boundary of FP8 may fall to its other side (a step is 1/16 or 1/8 of
        # the value); everything else is 32-bit sums and one rounding to bf16
        return {"rel": 6e-3, "max": 0.15}
    if case["kind"] == "producer":
        # values next to a rounding boundary of FP8 (a step is up to 1/8 of the value) or, postnorm, of bf16
        return {"rel": 2e-3, "max": 0.13}
    return {"rel": 6e-3, "max": 0.13}


# ---------------------------------------------------------------------------------------------- the same in 64 bits
def _scale64(x, fmt, basis=None):
    a = (x.abs().max().float() if basis is None else basis).reshape(1)
    return torch.full((1,), FP8_MAX[fmt], device="cuda") / a


def _codes64(x, rho, fmt):
    """FP8 codes of the saturating cast of rho * x (one binary32 product, round to nearest even)."""
    t = (x.float() * rho.float()).clamp_(-FP8_MAX[fmt], FP8_MAX[fmt])
    return t.to(FP8_DTYPE[fmt])


def _fp8_64(t, fmt):
    """float64 values rounded to the FP8 grid, saturating."""
    return t.float().clamp_(-FP8_MAX[fmt], FP8_MAX[fmt]).to(FP8_DTYPE[fmt]).double()


def _mm(a, b):
    return torch.mm(a.contiguous(), b.contiguous())


def _exact_linear(case, st):
    def cast(c):
        basis = torch.tensor(1.05, device="cuda") * c.x.abs().max().float() if case["scaling"] == "delayed" else None
        rho = _scale64(c.x, c.fmt, basis)
        q = _codes64(c.x, rho, c.fmt)
        return rho, q, q.double() / rho.double()
    sX, qX, X = cast(st["X"])
    sW, qW, W = cast(st["W"])
    out = {"Y": _mm(X, W.t()), "Xq": qX.view(torch.uint8), "Wq": qW.view(torch.uint8), "sX": sX.double(), "sW": sW.double()}
    if case["backward"]:
        sG, qG, G = cast(st["dY"])
        out.update(dX=_mm(G, W), dW=_mm(G.t(), X), dYq=qG.view(torch.uint8), sdY=sG.double())
        if case["scaling"] == "jit_transposed":
            out.update(XqT=qX.view(torch.uint8).t().contiguous(), dYqT=qG.view(torch.uint8).t().contiguous())
    return out


def _exact_attention(case, st):
    B, H, Hk, S, causal = case["B"], case["H"], case["H_kv"], case["S"], case["causal"]
    G = H // Hk
    val = {}
    for name in ("Q", "K", "V") + (("dO",) if case["backward"] else ()):
        c = st[name]
        if name in ("Q", "K") and case["producer"] != "jit":
            x = c.x.double()
            y = x / x.square().mean(dim=1, keepdim=True).sqrt() * GAIN if case["producer"] == "rmsnorm" else torch.tanh(ALPHA_T * x)
            rho = c.scale.double()
            val[name] = _fp8_64(y * rho, E4M3) / rho
        else:
            rho = _scale64(c.x, c.fmt)
            val[name] = _codes64(c.x, rho, c.fmt).double() / rho.double()
        val[name] = val[name].view(-1, S, HEAD_DIM)
    log2e = 1.4426950408889634
    O = torch.empty((B * H, S, HEAD_DIM), dtype=torch.float64, device="cuda")
    lse = torch.empty((B * H, S), dtype=torch.float64, device="cuda")
    dQ, dK, dV = torch.zeros_like(O), torch.zeros((B * Hk, S, HEAD_DIM), dtype=torch.float64, device="cuda"), torch.zeros((B * Hk, S, HEAD_DIM), dtype=torch.float64, device="cuda")
    amax_p = torch.zeros((), dtype=torch.float64, device="cuda")
    amax_ds = torch.zeros((), dtype=torch.float64, device="cuda")
    above = torch.ones((S, S), dtype=torch.bool, device="cuda").triu_(1) if causal else None
    dO_hi = st["dO"].x.double().view(-1, S, HEAD_DIM) if case["backward"] else None
    for bh in range(B * H):
        kv = bh // G
        q, k, v = val["Q"][bh], val["K"][kv], val["V"][kv]
        x = _mm(q, k.t()) * (st["s"] * log2e)
        if causal:
            x.masked_fill_(above, -math.inf)
        m = x.max(dim=1, keepdim=True).values.ceil()
        p = torch.exp2(x - m)
        l = p.sum(dim=1, keepdim=True)
        O[bh] = _mm(_fp8_64(448.0 * p, E4M3), v) / (448.0 * l)
        lse[bh] = (m + l.log2())[:, 0]
        amax_p = torch.maximum(amax_p, p.max())
        if case["backward"]:
            do = val["dO"][bh]
            P = torch.exp2(x - lse[bh][:, None])
            D = (dO_hi[bh] * O[bh].bfloat16().double()).sum(dim=1, keepdim=True)
            dV[kv] += _mm(_fp8_64(448.0 * P, E4M3).t(), do) / 448.0
            dS = P * (_mm(do, v.t()) - D)
            amax_ds = torch.maximum(amax_ds, dS.abs().max())
            dS = _fp8_64(SCALE_DS * dS, E5M2) / SCALE_DS
            dQ[bh] = _mm(dS, k) * st["s"]
            dK[kv] += _mm(dS.t(), q) * st["s"]
    out = {"O": O.view(-1, HEAD_DIM), "lse": lse.view(-1), "amax_p": amax_p.view(1)}
    if case["backward"]:
        out.update(dQ=dQ.view(-1, HEAD_DIM), dK=dK.view(-1, HEAD_DIM), dV=dV.view(-1, HEAD_DIM), amax_ds=amax_ds.view(1))
    return out


def _postnorm64(x, y, gamma):
    return x.double() + gamma.double() * y / y.square().mean(dim=1, keepdim=True).sqrt()


def _gelu64(x):
    return 0.5 * x * torch.erfc(-x / math.sqrt(2.0))


def _exact_producer(case, st):
    x, rho, op = st["x"].double(), st["scale"].double(), case["op"]
    if op == "postnorm":
        xnew = _postnorm64(x, st["y"].double(), st["gamma"])
        stored = xnew.to(torch.bfloat16)
        return {"xnew": xnew, "q": _codes64(stored, st["scale"], E4M3).double(), "amax": stored.abs().max().double().view(1)}
    if op == "rmsnorm":
        y = GAIN * x / x.square().mean(dim=1, keepdim=True).sqrt()
    elif op == "tanh":
        y = torch.tanh(ALPHA_T * x)
    elif op == "xielu":
        y = torch.where(x > 0, ALPHA_P * x * x + 0.5 * x, ALPHA_N * torch.expm1(x.clamp(max=0.0)) - ALPHA_N * x + 0.5 * x)
    else:
        y = _gelu64(x)
    return {"q": _fp8_64(y * rho, E4M3), "amax": y.abs().max().view(1)}


def _exact_ffn(case, st):
    def cast(c):
        rho = _scale64(c.x, c.fmt)
        return _codes64(c.x, rho, c.fmt).double() / rho.double()
    h = _mm(cast(st["X"]), cast(st["W1"]).t())
    a = _gelu64(h.to(torch.bfloat16).double())
    hq = _fp8_64(a * st["scale_h"].double(), E4M3)
    y = _mm(hq / st["scale_h"].double(), cast(st["W2"]).t())
    xnew = _postnorm64(st["X"].x, y.to(torch.bfloat16).double(), st["gamma"])
    stored = xnew.to(torch.bfloat16)
    return {"h": h, "hq": hq, "y": y, "xnew": xnew, "xq": _codes64(stored, st["scale_x"], E4M3).double(),
            "amax_h": a.abs().max().view(1), "amax_x": stored.abs().max().double().view(1)}


def exact(case, seed):
    """What run() returns, in 64 bits with plain torch (the FP8 casts that the path is defined by included)."""
    st = prepare(case, seed)
    return {"linear": _exact_linear, "attention": _exact_attention, "producer": _exact_producer, "ffn": _exact_ffn}[case["kind"]](case, st)
