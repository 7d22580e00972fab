"""GPU parity: QK RMS normalisation fused with the FP8 cast against the float64 oracle.

The normalised tensor is never stored, so a code is a rounding decision on a binary32 value; the
oracle gives, per element, the codes at both ends of a 2^-20 relative window.  Where they coincide
(all but a few elements in 10^5) the GPU byte must equal them; elsewhere it must be one of the two.
"""
import numpy as np
import pytest
import torch

from oracle import fp8, qknorm
from paper_2505_20524_amd import fog, synth
from parity import dev, fscalar, host_u16

pytestmark = pytest.mark.gpu


def run(xb, cols, fmt, rho, gain, pad_q=0):
    rows = xb.shape[0]
    x = dev(xb)
    if xb.shape[1] != cols:
        x = x[:, :cols]
    qfull = torch.full((rows, cols + pad_q), 0xAA, dtype=torch.uint8, device="cuda")
    q = qfull[:, :cols] if pad_q else qfull
    am = torch.full((1,), -1.0, device="cuda")
    fog.rmsnorm_quantize(x, fmt, fscalar(rho), q, gain=gain, amax_out=am)
    torch.cuda.synchronize()
    if pad_q:
        assert (qfull[:, cols:] == 0xAA).all()              # nothing written past the row
    return q.cpu().numpy(), am.item()


def check(xb, cols, fmt, rho, gain, pad_q=0):
    q, am = run(xb, cols, fmt, rho, gain, pad_q)
    view = xb[:, :cols]
    lo, hi = qknorm.quantize_window(view, rho, fmt, gain)
    undecided = lo != hi
    assert np.array_equal(q[~undecided], lo[~undecided])
    assert np.all((q[undecided] == lo[undecided]) | (q[undecided] == hi[undecided]))
    assert undecided.mean() <= 1e-3
    want = qknorm.amax(view, gain)
    assert abs(am - want) <= 2.0 ** -20 * want
    return q


@pytest.mark.parametrize("fmt", [fp8.E4M3, fp8.E5M2])
@pytest.mark.parametrize("rows,cols,pad", [(1, 128, 0), (4, 128, 0), (1000, 128, 0), (8192, 128, 0), (333, 64, 0), (100, 256, 8),
                                           (65, 512, 0), (50, 100, 0), (7, 17, 3), (129, 136, 0)])
def test_qknorm_parity(rows, cols, pad, fmt):
    rng = np.random.default_rng(rows + cols + fmt)
    x = rng.standard_normal((rows, cols + pad)).astype(np.float32) * 10.0 ** rng.uniform(-2, 2, (rows, 1))
    x[:, 1 % cols] *= 30.0                               # an outlier channel: the case the normalisation is there for
    xb = synth.f32_to_bf16_bits(x)
    gain = 1.0 if rows % 2 else 0.8
    rho = np.float32(fp8.fp8_max(fmt) / (gain * np.sqrt(cols)))      # the scale that cannot saturate
    check(xb, cols, fmt, rho, gain, pad_q=pad)


def test_qknorm_special_rows_and_saturation():
    D = 128
    x = np.zeros((6, D), np.float32)
    x[1, :] = 2.0                                         # constant: y = 1
    x[2, 40] = -3.0                                       # one-hot: y = -sqrt(D)
    x[3, ::2] = 1.0; x[3, 1::2] = -1.0
    x[4, :] = np.linspace(-1, 1, D)
    xb = synth.f32_to_bf16_bits(x)                        # rows 0 and 5 stay zero
    q = check(xb, D, fp8.E4M3, np.float32(448.0 / np.sqrt(D)), 1.0)
    assert not q[0].any() and not q[5].any()
    d = fp8.decode(q, fp8.E4M3)
    assert np.all(d[1] == d[1, 0]) and d[2, 40] < 0 and np.count_nonzero(d[2]) == 1
    # a scale four times too large: the one-hot element saturates at -448, nothing turns into NaN
    q = check(xb, D, fp8.E4M3, np.float32(4 * 448.0 / np.sqrt(D)), 1.0)
    assert fp8.decode(q, fp8.E4M3)[2, 40] == -448.0 and np.isfinite(fp8.decode(q, fp8.E4M3)).all()


def test_qknorm_several_trips_per_workgroup():
    """More rows than one trip of the largest grid covers (256 workgroups x 256 rows at D = 128): the pipelined
    loop runs several trips with a ragged last one; config 5's Q has 262144 rows."""
    rng = np.random.default_rng(11)
    rows = 3 * 131072 + 77
    xb = synth.f32_to_bf16_bits(rng.standard_normal((rows, 128)).astype(np.float32))
    check(xb, 128, fp8.E4M3, np.float32(448.0 / 5.0), 1.0)
    xb = synth.f32_to_bf16_bits(rng.standard_normal((2048 * 32 * 2 + 5, 64)).astype(np.float32))
    check(xb, 64, fp8.E5M2, np.float32(57344.0 / 5.0), 1.25)


def test_qknorm_config_shape_and_errors():
    """The Q tensor of config 3 whole ([B H S, 128] = 131072 rows), then the argument checks."""
    cfg = synth.CONFIGS[3]
    xb = synth.attention_tensors(cfg)["Q"].reshape(-1, 128)
    check(xb, 128, fp8.E4M3, np.float32(448.0 / np.sqrt(128)), 1.0)
    lib = fog.load()
    st = torch.cuda.current_stream().cuda_stream
    x = torch.zeros((4, 128), dtype=torch.int16, device="cuda")
    q = torch.zeros((4, 128), dtype=torch.uint8, device="cuda")
    f = fscalar(1.0)
    call = lib.fog_rmsnorm_quantize
    assert call(x.data_ptr(), 4, 128, 128, 1.0, 0, None, q.data_ptr(), 128, None, st) == 1
    assert call(x.data_ptr(), 4, 128, 128, 1.0, 0, f.data_ptr(), None, 128, None, st) == 1
    assert call(x.data_ptr(), 4, 128, 64, 1.0, 0, f.data_ptr(), q.data_ptr(), 128, None, st) == 2
    assert call(x.data_ptr(), -4, 128, 128, 1.0, 0, f.data_ptr(), q.data_ptr(), 128, None, st) == 2
    assert call(x.data_ptr() + 1, 4, 64, 64, 1.0, 0, f.data_ptr(), q.data_ptr(), 64, None, st) == 3
    assert call(x.data_ptr(), 4, 128, 128, 0.0, 0, f.data_ptr(), q.data_ptr(), 128, None, st) == 4
    assert call(x.data_ptr(), 4, 128, 128, 1.0, 3, f.data_ptr(), q.data_ptr(), 128, None, st) == 4
    assert call(None, 0, 128, 128, 1.0, 0, f.data_ptr(), None, 128, f.data_ptr(), st) == 0
    torch.cuda.synchronize()
    assert f.item() == 0.0                                 # the abs-max of an empty tensor is written as 0


@pytest.mark.parametrize("fmt", [fp8.E4M3, fp8.E5M2])
@pytest.mark.parametrize("rho", [39.0, 3.0e38, float("nan")])
def test_qknorm_special_values_take_the_careful_cast(rho, fmt):
    """Rows that hold NaN, infinities or values whose squares overflow, and scales that overflow every product or are NaN: the
    rows kernel (which casts without clamp or NaN test where it can) against the general kernel, which has no such form.  Ordinary
    rows under an ordinary scale may differ in the last bit of the norm, all others agree to the byte."""
    D, rows = 128, 70
    rng = np.random.default_rng(8)
    x = rng.standard_normal((rows, D)).astype(np.float32)
    x[3, 5], x[9, 7], x[9, 8], x[20, 1], x[33, 100], x[40] = np.nan, np.inf, 1.0, -np.inf, 3e38, 0.0
    x[41, :2] = (-np.nan, np.inf)
    xd = dev(synth.f32_to_bf16_bits(np.where(np.isnan(x), 0, x)))
    bits = xd.cpu().numpy().view(np.uint16).copy()
    bits[3, 5], bits[41, 0] = 0x7FC1, 0xFFC1
    xd = dev(bits)
    out = []
    for pad in (0, 1):
        q = torch.zeros((rows, D + pad), dtype=torch.uint8, device="cuda")[:, :D]
        am = torch.zeros(1, device="cuda")
        fog.rmsnorm_quantize(xd, fmt, fscalar(rho), q, amax_out=am)
        torch.cuda.synchronize()
        out.append((q.cpu().numpy(), am.item()))
    special = [3, 9, 20, 33, 40, 41]
    assert np.array_equal(out[0][0][special], out[1][0][special])
    if rho == 39.0:
        assert (out[0][0] != out[1][0]).mean() < 1e-3
    else:
        assert np.array_equal(out[0][0], out[1][0])
    assert np.isnan(out[0][1]) and np.isnan(out[1][1])


@pytest.mark.parametrize("fmt", [fp8.E4M3, fp8.E5M2])
@pytest.mark.parametrize("cols", [128, 512])
@pytest.mark.parametrize("gain,rho", [(1.0, 39.0), (1.0e30, 1.0e-30), (3.0e38, 1.0e-10)])
def test_qknorm_norm_or_product_beyond_binary32(gain, rho, cols, fmt):
    """Finite rows whose inverse norm is not finite (squares so small that their mean rounds to 0, a gain over a small norm) and
    gains whose product with an element overflows: the rows kernel gives the bytes and the abs-max of the general kernel, which
    clamps every element, and what is not zero saturates."""
    rows = 70
    rng = np.random.default_rng(9)
    x = rng.standard_normal((rows, cols)).astype(np.float32)
    x[2], x[5], x[9] = 0.0, 0.0, 0.0
    x[2, 17] = 2.0 ** -74                                             # its square / cols is below half the smallest subnormal
    x[5, 40:80] = 1.25 * 2.0 ** -75 * rng.choice([-1.0, 1.0], 40)     # each square rounds up to one subnormal step
    x[9, [3, 4, 60, 127]] = (1e-22, -1e-22, 1e-22, 1e-22)
    x[12] *= np.float32(1e-10)                                        # gain 1e30 over a norm of 1e-10
    xd = dev(synth.f32_to_bf16_bits(x))
    nonzero = synth.bf16_bits_to_f32(host_u16(xd)) != 0
    top = 0x7E if fmt == fp8.E4M3 else 0x7B
    out = []
    for pad in (0, 1):                 # an odd ldq takes the general kernel
        q = torch.zeros((rows, cols + pad), dtype=torch.uint8, device="cuda")[:, :cols]
        am = torch.zeros(1, device="cuda")
        fog.rmsnorm_quantize(xd, fmt, fscalar(rho), q, gain=gain, amax_out=am)
        torch.cuda.synchronize()
        out.append((q.cpu().numpy(), am.item()))
    special = [2, 5, 9] if gain == 1.0 else [2, 5, 9, 12] if gain == 1.0e30 else list(range(rows))
    got, want = out[0][0], out[1][0]
    assert np.array_equal(got[special], want[special])
    assert (got != want).mean() < 1e-3                                # ordinary rows: the last bit of the norm, as elsewhere
    for r in special:
        assert ((got[r] & 0x7F)[nonzero[r]] == top).all()
    assert np.isnan(out[0][1]) and np.isnan(out[1][1])                # zero times an infinite inverse norm


@pytest.mark.parametrize("rows,cols", [(8191, 128), (8192, 128), (16383, 64), (4097, 256), (2047, 512), (262145, 128), (524289, 128)])
def test_every_form_gives_the_rows_of_small_calls(rows, cols):
    """Workgroups of 256 and of 1024 threads, ordinary and non-temporal loads: the bytes and the abs-max that calls of 96 rows give."""
    g = torch.Generator(device="cuda").manual_seed(rows)
    x, rho = torch.randn((rows, cols), device="cuda", generator=g).to(torch.bfloat16), fscalar(39.0)
    q, am, largest = torch.zeros((rows, cols), dtype=torch.uint8, device="cuda"), torch.full((1,), -1.0, device="cuda"), 0.0
    fog.rmsnorm_quantize(x, fp8.E4M3, rho, q, amax_out=am)
    top = int((x.abs().amax(dim=1).float() / x.float().square().mean(dim=1).sqrt()).argmax())   # the row that holds the largest result
    for first in sorted({0, 96 * 20, top // 96 * 96, (rows - 1) // 96 * 96}):
        part = slice(first, min(first + 96, rows))
        want, wam = torch.zeros((part.stop - first, cols), dtype=torch.uint8, device="cuda"), torch.zeros(1, device="cuda")
        fog.rmsnorm_quantize(x[part], fp8.E4M3, rho, want, amax_out=wam)
        assert torch.equal(q[part], want)
        largest = max(largest, wam.item())
    assert am.item() == largest
