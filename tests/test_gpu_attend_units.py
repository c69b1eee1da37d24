"""The attention kernel's units of 32 keys (Alg. 1 steps 4-5): lists of 0 to 6 blocks whose last block is ragged at either half
of it, and query blocks that end in either half of their rows, with logits that pass the range of the fp16 weights in every unit
(each is formed again with a raised reference), in some or in none, in every form of the kernel, against the oracle on the fp32 result."""
import numpy as np
import pytest

from paper_2605_11354_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _run(oracle, bq, dtype, launch, tail, binades, scales=(0,)):
    """(result, reference [query block, row, channel], largest |V| of the query block's list) with exponents rising by `binades` from
    unit to unit and values of 2^scales[j % ..] in block j."""
    rng = np.random.default_rng(100 * tail + binades)
    nkb = 13
    N = (nkb - 1) * 64 + tail
    c = 0.125 * np.log2(np.e)
    q, k, v = (rng.standard_normal((N, 64)) for _ in range(3))
    v *= 2.0 ** np.array(scales, float)[np.arange(N) // 64 % len(scales), None]
    q += 1.0                                           # (spread over the channels: the E4M3 unit aligns a product's terms to the largest)
    k += ((np.arange(N) // 32) * binades / (64.0 * c))[:, None]
    cfg = synth.CONFIGS[1].with_(B=1, H=1, N=N, bq=bq, dtype=dtype, proj_per_head=False)
    d = {"Q": synth.to_bf16_bits(q)[None, None], "K": synth.to_bf16_bits(k)[None, None], "V": synth.to_bf16_bits(v)[None, None],
         "W": synth.to_bf16_bits(np.eye(64))[None], "sQ": None, "sK": None, "sV": None}
    if dtype == "fp8":
        for t, blk in (("Q", bq), ("K", 64), ("V", 64)):
            d[t], d["s" + t] = synth.quantise_e4m3_blocks(d[t], blk)
    case = G.Case(cfg, {n: None if a is None else np.ascontiguousarray(a) for n, a in d.items()}, k_crit=6, k_neg=0)
    lab = np.zeros((1, 1, case.Nqb, nkb), np.int8)
    top = np.zeros(case.Nqb)
    for i in range(case.Nqb):
        n = i % 7
        js = np.sort(rng.choice(nkb - 1, n, replace=False))
        if n and i % 2:
            js[-1] = nkb - 1                           # with the ragged block
        lab[0, 0, i, js] = 2
        top[i] = max([np.abs(v[64 * j:64 * j + 64]).max() for j in js], default=0.0)
    O = G.sparse_f32(case, lab, launch)
    ref = case.oracle_attend(oracle, lab, want_parts=True)
    return G.gather_blocks(O[None, None], ref["sel"], bq, 1), ref["O_sparse"], top


@pytest.mark.parametrize("bq,dtype,launch", G.ATTEND_FORMS)
@pytest.mark.parametrize("tail", [1, 31, 32, 33, 64])
@pytest.mark.parametrize("binades", [0, 7, 20])        # by which a unit's exponents lie above those of the one before
def test_ragged_units_and_raised_references(oracle, bq, dtype, launch, tail, binades):
    got, want, _ = _run(oracle, bq, dtype, launch, tail, binades)
    err = np.abs(got - want).max() / np.sqrt(np.mean(want ** 2))
    print(f"bq={bq} {dtype} {launch} tail={tail} binades={binades}: {err:.3e}")
    # fp16 weights: 2^-11 each on sums that cancel to a few times that; logits of up to 520 binades: 520 x 2^-24 at each of a few
    # roundings, below 2^-12 of a weight
    assert err <= 2.0 ** -8


@pytest.mark.parametrize("bq,dtype,launch", G.ATTEND_FORMS)
@pytest.mark.parametrize("tail", [1, 33, 64])
@pytest.mark.parametrize("binades", [0, 7, 20])
@pytest.mark.parametrize("scales", [(0, -10, 12, -3, 30), (30, 0, -70), (-9, 9)])       # within and beyond what the row sums' factor holds
def test_raised_references_and_far_scales(oracle, bq, dtype, launch, tail, binades, scales):
    """An output is a convex combination of its list's values.  Its weights are off by 2^-11 (fp16) and 2^-12 (logits, as above), so it
    is off by at most the sum of the two times the largest of those values, in the numerator and again in the row sums."""
    got, want, top = _run(oracle, bq, dtype, launch, tail, binades, scales)
    err = (np.abs(got - want).max(axis=(1, 2)) / np.maximum(top, 1e-30))[top > 0].max()
    print(f"bq={bq} {dtype} {launch} tail={tail} binades={binades} {scales}: {err:.3e}")
    assert err <= 2 * (2.0 ** -11 + 2.0 ** -12)
