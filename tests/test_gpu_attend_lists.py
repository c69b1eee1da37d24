"""The attention kernel's forms of an iteration (Alg. 1 steps 4-5): list lengths around the points where the guard-free
iterations begin and end and where the window of 64 entries moves, with logits that hardly ever pass the first unit's maximum by the
2^12 that a weight may grow, and with logits that do so often, against the oracle on the fp32 result."""
import numpy as np
import pytest
import torch

from paper_2605_11354_amd import binding as B
from paper_2605_11354_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bq,dtype", [(64, "bf16"), (128, "bf16"), (64, "fp8"), (128, "fp8")])
@pytest.mark.parametrize("gain", [1.0, 1.3, 5.0])      # of K: the reference is hardly ever, sometimes, often raised
def test_list_lengths_and_raised_references(oracle, bq, dtype, gain):
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
    O = torch.full((1, 1, cfg.N, 64), float("nan"), dtype=torch.float32, device="cuda")
    B.sla_sparse_combine_f32(case.p, case.Q, case.K, case.V, None, torch.from_numpy(lab).cuda(), None, O, case.sQ, case.sK, case.sV, case.ws)
    torch.cuda.synchronize()
    ref = case.oracle_attend(oracle, lab, want_parts=True)
    got = G.gather_blocks(O.cpu().numpy().astype(np.float64), ref["sel"], bq, 1)
    err = np.abs(got - ref["O_sparse"]).max() / np.sqrt(np.mean(ref["O_sparse"] ** 2))
    print(f"bq={bq} {dtype} gain={gain}: {err:.3e}")
    assert err <= G.TOL[dtype]                                    # the stated bar, on the result before the bf16 store
