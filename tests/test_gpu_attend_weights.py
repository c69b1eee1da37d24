"""The softmax weights of the attention kernel (Alg. 1 steps 4-5) where 16 bits could lose them, against the oracle on the
fp32 result, in every form of the kernel: rows with one dominant key of no value, long lists whose keys grow from one window of
64 entries to the next in directions the queries do not see, and blocks of values of very different size."""
import numpy as np
import pytest
import torch

from paper_2605_11354_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _case(q, k, v, bq, dtype):
    """Every key block critical.  q, k, v: float [N,64]."""
    N = q.shape[0]
    cfg = synth.CONFIGS[1].with_(B=1, H=1, N=N, bq=bq, dtype=dtype, proj_per_head=False)
    d = {"Q": synth.to_bf16_bits(q)[None, None], "K": synth.to_bf16_bits(k)[None, None], "V": synth.to_bf16_bits(v)[None, None],
         "W": synth.to_bf16_bits(np.eye(64))[None], "sQ": None, "sK": None, "sV": None}
    if dtype == "fp8":
        for t, blk in (("Q", bq), ("K", 64), ("V", 64)):
            d[t], d["s" + t] = synth.quantise_e4m3_blocks(d[t], blk)
    d = {n: None if a is None else np.ascontiguousarray(a) for n, a in d.items()}
    Nkb = -(-N // 64)
    return G.Case(cfg, d, k_crit=Nkb, k_neg=0)


def _error(case, oracle, lab, sel, launch=0):
    """Largest error of the sparse output over the blocks of sel, relative to its RMS."""
    ref = case.oracle_attend(oracle, lab, sel=sel, want_parts=True)
    got = G.gather_blocks(G.sparse_f32(case, lab, launch)[None, None], sel, case.cfg.bq, 1)
    return float(np.abs(got - ref["O_sparse"]).max() / np.sqrt(np.mean(ref["O_sparse"] ** 2)))


@pytest.mark.parametrize("bq,launch", [(64, 0), (128, 0), (128, 769)])
@pytest.mark.parametrize("above", [1.0, 3.0, 4.5])      # of |q| max|k| over the largest exponent plus 15, in binades
def test_small_weights_under_a_dominant_key(oracle, bq, launch, above):
    """A key of zero V at exponent 17, all others near 2^-17 of its weight: fp16 holds such weights in steps of 2^-24 of the
    largest, an error of at most 2^-25 each.  Uniform errors on n weights against the weights' own 2-norm (at least
    2^-17 sqrt(n)): 2^-25 / sqrt(3) / 2^-17 = 2.3e-3 RMS, five times that for the largest of 140000 values, and the weights
    above 2^-14, in whole fp16 precision, add 2^-11 at most.  A reference some binades above the largest weight multiplies
    the first by two for each of them."""
    rng = np.random.default_rng(int(above) + bq)
    N, c = 34 * 64, 0.125 * np.log2(np.e)
    q = np.zeros((N, 64))
    q[:, 0] = 8.0
    peak = 17.0 / (8.0 * c)
    k = np.zeros((N, 64))
    k[:, 0] = (0.0 + rng.standard_normal(N)) / (8.0 * c)
    k[7, 0] = peak
    side = rng.standard_normal((N, 63))
    length = (17.0 + 15.0 + above) / (8.0 * c)
    k[:, 1:] = side / np.linalg.norm(side, axis=1, keepdims=True) * np.sqrt(length ** 2 - k[:, :1] ** 2)
    v = rng.standard_normal((N, 64))
    v[7] = 0.0
    case = _case(q, k, v, bq, "bf16")
    lab = np.full((1, 1, case.Nqb, case.Nkb), 2, np.int8)
    err = _error(case, oracle, lab, [(0, 0), (0, case.Nqb - 1)], launch)
    print(f"bq={bq} {launch} above={above}: {err:.3e}")
    assert err <= 1.2e-2


@pytest.mark.parametrize("bq,dtype,launch", G.ATTEND_FORMS)
def test_keys_that_grow_along_the_list(oracle, bq, dtype, launch):
    """256 critical blocks, |k| growing by a quarter every 32 blocks in channels where q is zero, logits near zero: all keys
    weigh about the same.  Values of 1 in the last 64 blocks and of 1/4 before, so that the output tells their share of the
    weight."""
    rng = np.random.default_rng(bq)
    N, c = 256 * 64, 0.125 * np.log2(np.e)
    q = np.zeros((N, 64))
    q[:, :8] = rng.standard_normal((N, 8))
    q[:, :8] *= 8.0 / np.linalg.norm(q[:, :8], axis=1, keepdims=True)
    k = np.zeros((N, 64))
    k[:, :8] = 0.2 * rng.standard_normal((N, 8))
    side = rng.standard_normal((N, 56))
    length = 14.0 + 3.8 * np.maximum(np.arange(N) // 2048 - 1, 0)
    k[:, 8:] = side / np.linalg.norm(side, axis=1, keepdims=True) * length[:, None]
    v = np.full((N, 64), 0.25)
    v[192 * 64:] = 1.0
    case = _case(q, k, v, bq, dtype)
    lab = np.full((1, 1, case.Nqb, case.Nkb), 2, np.int8)
    err = _error(case, oracle, lab, [(0, 0), (0, case.Nqb - 1)], launch)
    print(f"bq={bq} {dtype} {launch}: {err:.3e}")
    assert err <= 2e-3                                   # fp16 weights (2^-11) on a sum that cancels nothing


@pytest.mark.parametrize("bq,dtype,launch", G.ATTEND_FORMS)
@pytest.mark.parametrize("length,zeros", [(2, [0]), (2, [0, 1]), (5, [0]), (5, [2, 4]), (9, [0, 1, 2, 8]), (70, list(range(66)))])
def test_blocks_of_zero_values(oracle, bq, dtype, launch, length, zeros):
    """Key blocks whose V is zero weigh like any other, also at the head of a list (positions `zeros` of the list)."""
    rng = np.random.default_rng(length)
    nkb = 72
    q, k, v = (rng.standard_normal((nkb * 64 - 5, 64)) for _ in range(3))
    js = np.sort(rng.choice(nkb - 1, length, replace=False))
    for z in zeros:
        v[64 * js[z]:64 * js[z] + 64] = 0.0
    case = _case(q, k, v, bq, dtype)
    case.p.k_crit, case.p.k_neg = length, 0
    lab = np.zeros((1, 1, case.Nqb, case.Nkb), np.int8)
    lab[..., js] = 2
    sel = [(0, 0), (0, case.Nqb - 1)]
    ref = case.oracle_attend(oracle, lab, sel=sel, want_parts=True)["O_sparse"]
    got = G.gather_blocks(G.sparse_f32(case, lab, launch)[None, None], sel, bq, 1)
    err = np.abs(got - ref).max() / max(np.sqrt(np.mean(ref ** 2)), 1e-3)
    print(f"bq={bq} {dtype} {launch} {length} {zeros[-1]}: {err:.3e}")
    assert err <= 2.0 ** -8                                 # fp16 weights, 2^-11, on sums whose terms cancel to a few times that


@pytest.mark.parametrize("bq,dtype,launch", G.ATTEND_FORMS)
@pytest.mark.parametrize("scales", [(-17, 0), (-12, 0), (0, -12), (0, 12, 0, -5, 6)])
def test_values_of_far_apart_scales(oracle, bq, dtype, launch, scales):
    """Values of 2^scales[i % ...] in block i: a block of small values counts in the sums whatever stands in front of it."""
    rng = np.random.default_rng(len(scales))
    nkb = 72
    q, k, v = (rng.standard_normal((nkb * 64 - 5, 64)) for _ in range(3))
    v *= 2.0 ** np.array(scales, float)[np.arange(len(v)) // 64 % len(scales), None]
    case = _case(q, k, v, bq, dtype)
    lab = np.full((1, 1, case.Nqb, case.Nkb), 2, np.int8)
    lab[0, 0, 0, 9:] = 0                                    # a short list and the whole of it
    case.p.k_crit = nkb
    err = max(_error(case, oracle, lab, [(0, 0)], launch), _error(case, oracle, lab, [(0, case.Nqb - 1)], launch))
    print(f"bq={bq} {dtype} {launch} {scales}: {err:.3e}")
    assert err <= 2.0 ** -8


@pytest.mark.parametrize("bq,dtype,launch", G.ATTEND_FORMS)
@pytest.mark.parametrize("scales", [(0, -120), (2, -126), (90, -40), (0, -60), (-120, 0), (-126, 2), (-40, 90), (2, -126, -126, 2, -60)])
@pytest.mark.parametrize("tail", [64, 40])             # tokens of the last block
def test_values_at_the_ends_of_the_range(oracle, bq, dtype, launch, scales, tail):
    """Values of 2^scales[j] in block j, up to the whole range of bf16 apart and in either order, two blocks (the short-list
    kernel with 64-row query blocks) and five: a block whose values vanish beside another's still takes its share of the weight."""
    rng = np.random.default_rng(len(scales) + tail)
    N = 64 * len(scales) - 64 + tail
    q, k, v = (rng.standard_normal((N, 64)) for _ in range(3))
    v = v * np.float32(2.0) ** np.repeat(np.array(scales, np.float32), 64)[:N, None]
    case = _case(q, k, v, bq, "bf16")
    u = np.ascontiguousarray(v, dtype=np.float32).view(np.uint32)          # (values below 2^-20 stay)
    d = dict(case.d, V=((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)[None, None])
    if dtype == "fp8":
        for t, blk in (("Q", bq), ("K", 64), ("V", 64)):
            d[t], d["s" + t] = synth.quantise_e4m3_blocks(d[t], blk)
    case = G.Case(case.cfg.with_(dtype=dtype), {n: None if a is None else np.ascontiguousarray(a) for n, a in d.items()}, k_crit=len(scales), k_neg=0)
    lab = np.full((1, 1, case.Nqb, case.Nkb), 2, np.int8)
    err = _error(case, oracle, lab, [(0, i) for i in range(case.Nqb)], launch)
    print(f"bq={bq} {dtype} {launch} {scales} {tail}: {err:.3e}")
    assert err <= 2.0 ** -8                                 # fp16 weights, 2^-11, on sums whose terms cancel to a few times that


@pytest.mark.parametrize("bq,launch", [(64, 0), (128, 0), (128, 769)])
@pytest.mark.parametrize("nkb", [2, 9, 20])
def test_e4m3_block_scales_cancel(bq, launch, nkb):
    """Every query sees one key 184 binades above all others: its output is that key's V row, code times block scale.  The weight carries
    the scale relative to the list's and the row sum has it divided out again: what that leaves is below 2^-15 (two of fp16's roundings
    in turn, 2^-22, and a few of fp32), where a factor rounded to fp16 would leave up to 2^-12."""
    rng = np.random.default_rng(nkb)
    N = nkb * 64
    of_row = rng.integers(0, 32, N)
    key = 64 * (np.arange(32) % nkb) + rng.integers(0, 64, 32)
    q, k = np.zeros((N, 64)), np.zeros((N, 64))
    q[np.arange(N), of_row] = 32.0
    k[key, np.arange(32)] = 32.0
    v = rng.standard_normal((N, 64)) * np.repeat(rng.uniform(0.125, 8.0, nkb), 64)[:, None]
    case = _case(q, k, v, bq, "fp8")
    lab = np.full((1, 1, case.Nqb, case.Nkb), 2, np.int8)
    got = G.sparse_f32(case, lab, launch)
    codes = torch.from_numpy(case.d["V"][0, 0]).view(torch.float8_e4m3fn).double().numpy()
    want = (codes * np.repeat(case.d["sV"][0, 0].astype(np.float64), 64)[:, None])[key[of_row]]
    err = np.abs(got - want).max(axis=1) / np.abs(want).max(axis=1)
    print(f"bq={bq} {launch} {nkb}: {err.max():.3e}")
    assert err.max() <= 2.0 ** -15
