"""The attention kernel's lists (Alg. 1 steps 4-5): lengths around the points where the window of 64 entries moves (an iteration
reads two entries ahead of its own, the window moves by 32), odd and even (iterations run in pairs), with logits whose weights never (gains
1 and 1.3), now and then and often add up to more than the 2^15 per unit above which the reference is raised, in every form of the
kernel, against the oracle on the fp32 result."""
import numpy as np
import pytest

from paper_2605_11354_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bq,dtype,launch", G.ATTEND_FORMS)
@pytest.mark.parametrize("gain", [1.0, 1.3, 5.0, 15.0])      # of K
def test_list_lengths_and_raised_references(oracle, bq, dtype, launch, gain):
    cfg = synth.CONFIGS[1].with_(H=1, N=75 * 64 - 9, bq=bq)
    d = dict(synth.make_inputs(cfg))
    k = (d["K"].astype(np.uint32) << 16).view(np.float32) * np.float32(gain)
    d["K"] = synth.to_bf16_bits(k)
    if dtype == "fp8":
        cfg = cfg.with_(dtype="fp8")
        for t, blk in (("Q", bq), ("K", 64), ("V", 64)):
            d[t], d["s" + t] = synth.quantise_e4m3_blocks(d[t], blk)
    rng = np.random.default_rng(3)
    case = G.Case(cfg, d, k_crit=75, k_neg=0)
    lengths = [3, 4, 5, 6, 7, 9, 10, 33, 34, 61, 62, 63, 64, 65, 66, 68, 75]      # one per query block, ragged last block in and out
    lab = np.zeros((1, 1, case.Nqb, 75), np.int8)
    for i in range(case.Nqb):
        n = lengths[i % len(lengths)]
        js = rng.choice(75 if i % 2 or n == 75 else 74, n, replace=False)
        lab[0, 0, i, js] = 2
    O = G.sparse_f32(case, lab, launch)
    ref = case.oracle_attend(oracle, lab, want_parts=True)
    got = G.gather_blocks(O[None, None], ref["sel"], bq, 1)
    err = np.abs(got - ref["O_sparse"]).max() / np.sqrt(np.mean(ref["O_sparse"] ** 2))
    print(f"bq={bq} {dtype} {launch} gain={gain}: {err:.3e}")
    assert err <= G.TOL[dtype]                                    # the stated bar, on the result before the bf16 store
