"""The FP8 layer where the form of its two launches changes (rows that do not fill a group of 32, one and two passes over a
row, the last workgroup's half group, the three token tiles, the fewest K steps), and the quantisers' division step on
infinities, NaN and very large operands, against the oracle or the stated formula (App. B.2: scale = max(amax, 1e-8) / 448, IEEE division,
clamp, cast)."""
import numpy as np
import pytest
import torch

from paper_2605_11354_amd import binding as B
from paper_2605_11354_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d_in,d_out", [(1, 128, 8),                     # one row, one partial group of channels, two K steps
                                          (33, 1152, 72), (31, 2176, 264),  # slices held by fewer than four waves; two passes
                                          (65, 2048, 136), (16000, 1152, 384),     # one row in the last group, whole groups; 8 slices a wave
                                          (4100, 256, 2048),               # 128-token tiles, four rows in the last one
                                          (8195, 128, 2056), (8200, 384, 2048)])   # 256-token tiles, two and six K steps
def test_layer_at_the_edges_of_its_launches(oracle, N, d_in, d_out):
    rng = np.random.default_rng(N)
    xb = synth.to_bf16_bits((rng.standard_normal((N, d_in)) * np.exp(rng.uniform(-2, 2, (N, 1)))).astype(np.float32))
    Wb = synth.to_bf16_bits((rng.standard_normal((d_out, d_in)) / np.sqrt(d_in)).astype(np.float32))
    bb = synth.to_bf16_bits(rng.standard_normal(d_out).astype(np.float32))
    y = torch.full((N, d_out), float("nan"), dtype=torch.bfloat16, device="cuda")
    up = lambda n: -(-n // 256) * 256
    need = up(N * d_in) + up(4 * N) + up(d_out * d_in) + up(4 * d_out)
    ws = torch.full((need + 256,), 0x5A, dtype=torch.uint8, device="cuda")
    B.sla_fp8_linear(G.dev_bf16(xb), G.dev_bf16(Wb), G.dev_bf16(bb), y, ws[:-256])
    torch.cuda.synchronize()
    assert (ws[-256:] == 0x5A).all()
    ref = oracle.fp8_linear(xb, Wb, bb)
    got = G.bf16_tensor_to_f64(y)
    # codes and scales are the oracle's bit for bit; beyond the bf16 store there are d_in fp32 additions of exact products and
    # three roundings: |error| <= (d_in + 3) 2^-24 sum |x w|, and the sum of magnitudes stays below sqrt(d_in) RMS here
    rms = float(np.sqrt(np.mean(ref ** 2)))
    excess = np.maximum(np.abs(got - ref) - G.bf16_half_ulp(ref), 0.0).max() / rms
    assert excess <= max(1e-3, (d_in + 3) * 2.0 ** -24 * np.sqrt(d_in)), excess


def test_codes_of_infinities_and_nan():
    inf, nan = float("inf"), float("nan")
    x = torch.randn((1, 1, 192, 64), device="cuda").to(torch.bfloat16)
    x[0, 0, 5, 7], x[0, 0, 6, 1] = inf, nan          # block 0: infinite scale: finite -> zero of its sign, inf and NaN -> code of -448
    x[0, 0, 8], x[0, 0, 71], x[0, 0, 72] = -0.0, -0.0, 0.0
    x[0, 0, 70, 3] = nan                             # block 1: NaN does not count for the maximum
    codes = torch.empty(x.shape, dtype=torch.uint8, device="cuda")
    scales = torch.empty((1, 1, 3), dtype=torch.float32, device="cuda")
    B.sla_quantise_e4m3(x, 64, codes, scales)
    torch.cuda.synchronize()
    xf, c, s = x.float().cpu().numpy()[0, 0].reshape(3, 64, 64), codes.cpu().numpy()[0, 0].reshape(3, 64, 64), scales.cpu().numpy()[0, 0]
    assert np.isinf(s[0]) and s[1] == np.nanmax(np.abs(xf[1])) / np.float32(448) and s[2] == np.abs(xf[2]).max() / np.float32(448)
    want = np.where(np.isfinite(xf[0]), np.where(np.signbit(xf[0]), 0x80, 0), 0xFE)
    assert np.array_equal(c[0], want)
    q = np.clip(xf[1:] / s[1:, None, None], np.float32(-448), np.float32(448))
    q = torch.from_numpy(np.where(np.isnan(q), np.float32(-448), q)).to(torch.float8_e4m3fn).view(torch.uint8).numpy()
    assert np.array_equal(c[1:], q)


@pytest.mark.parametrize("N,d_in,d_out", [(40, 256, 72), (4100, 256, 2048), (8200, 384, 2048)])     # the three token tiles
@pytest.mark.parametrize("size_x,size_W", [(1e36, 1e-6), (1e-6, 1e36)])
def test_layer_on_very_large_operands(oracle, N, d_in, d_out, size_x, size_W):
    """The scale of one operand alone is far outside the range of y: no step on the way to a finite y overflows."""
    rng = np.random.default_rng(N)
    bits = lambda a: (np.ascontiguousarray(a, np.float32).view(np.uint32) >> 16).astype(np.uint16)       # (truncated: nothing flushed)
    xb, Wb = bits(rng.standard_normal((N, d_in)) * size_x), bits(rng.standard_normal((d_out, d_in)) * size_W)
    y = torch.full((N, d_out), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.sla_fp8_linear(G.dev_bf16(xb), G.dev_bf16(Wb), None, y)
    torch.cuda.synchronize()
    ref, got = oracle.fp8_linear(xb, Wb, None), G.bf16_tensor_to_f64(y)
    rms = float(np.sqrt(np.mean(ref ** 2)))
    excess = np.maximum(np.abs(got - ref) - G.bf16_half_ulp(ref), 0.0).max() / rms
    assert excess <= max(1e-3, (d_in + 3) * 2.0 ** -24 * np.sqrt(d_in)), excess
