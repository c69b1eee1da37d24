"""Rows of at most 64 key blocks (frame attention) where the short-row classifier and the states pass change form: one token,
one key block, 32 / 33 and 64 / 65 key blocks, ragged ends, rows of the last workgroup past the end, both query block sizes and
data types, ties; block means, logits, labels and critical lists bit for bit against the oracle, the result within its bar."""
import numpy as np
import pytest
import torch

from paper_2605_11354_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _variants(cfg, d):
    """plain; key blocks equal in pairs, every third pair apart by one tiny element; Q = 0 (all tie); a run of blocks of one
    tiny element each, of either sign (logits next to zero that differ in sign and exponent, or not at all)."""
    yield "plain", d
    K, whole = d["K"].copy(), cfg.N // 64
    for j in range(1, whole, 2):
        K[:, :, j * 64:(j + 1) * 64] = K[:, :, (j - 1) * 64:j * 64]
        if j % 3 == 0:
            K[:, :, j * 64 + 5, 3] = synth.to_bf16_bits(np.float32([2.0 ** -38]))[0]
    yield "pairs", dict(d, K=K)
    yield "all_tie", dict(d, Q=np.zeros_like(d["Q"]))
    K = d["K"].copy()
    for j in range(whole // 3, whole):
        K[:, :, j * 64:(j + 1) * 64] = 0
        K[:, :, j * 64, 3] = synth.to_bf16_bits(np.float32([(-1.0) ** j * 2.0 ** -(40 + j % 5)]))[0]
    yield "tiny", dict(d, K=K)


def _check(oracle, case, what):
    got, ref = case.classify(), case.oracle_classify(oracle, want_scores=True, want_pc=True, want_means=True)
    assert np.array_equal(got["labels"], ref["labels"]), what
    assert np.array_equal(got["qbar"], ref["qbar"]) and np.array_equal(got["kbar"], ref["kbar"]), what
    assert np.array_equal(got["scores"], ref["scores"]), what
    np.testing.assert_allclose(got["Pc"], ref["Pc"], rtol=2e-5, atol=1e-12, err_msg=str(what))      # fp32 exponentials
    if case.k_c:
        for idx in np.ndindex(got["labels"].shape[:3]):
            assert np.array_equal(got["crit_idx"][idx], np.nonzero(ref["labels"][idx] == 2)[0]), (what, idx)
    O, lab = case.forward()
    assert np.array_equal(lab.cpu().numpy(), ref["labels"]), what
    att = case.oracle_attend(oracle, ref["labels"])
    G.assert_output(G.gather_blocks(G.bf16_tensor_to_f64(O), att["sel"], case.cfg.bq, case.cfg.H), att["O"], case.cfg.dtype, str(what))


@pytest.mark.parametrize("Bn,H,N,bq,dtype", [(1, 1, 1, 64, "bf16"), (2, 3, 63, 128, "fp8"), (1, 2, 65, 64, "fp8"), (3, 2, 64 * 5 + 1, 128, "bf16"),
                                             (1, 2, 2048, 64, "bf16"), (1, 2, 2049, 64, "fp8"), (1, 1, 4096, 128, "bf16"),
                                             (1, 1, 4096, 64, "fp8"), (1, 1, 4097, 64, "bf16")])
def test_short_rows_at_their_edges(oracle, Bn, H, N, bq, dtype):
    cfg = synth.CONFIGS[4 if dtype == "fp8" else 0].with_(B=Bn, H=H, N=N, bq=bq, crit_frac=0.06, neg_frac=0.5, n_clusters=8)
    _check(oracle, G.Case(cfg), (Bn, H, N, bq, dtype))


@pytest.mark.parametrize("nkb,kc,kn", [(1, 1, 0), (1, 0, 1), (22, 2, 13), (32, 5, 20), (33, 0, 30), (64, 7, 0), (64, 64, 0)])
def test_short_rows_with_ties_and_extreme_counts(oracle, nkb, kc, kn):
    cfg = synth.CONFIGS[0].with_(H=2, N=nkb * 64 - 17, bq=64, n_clusters=16)
    for name, dd in _variants(cfg, synth.make_inputs(cfg)):
        case = G.Case(cfg, dd, k_crit=kc, k_neg=kn)
        got, ref = case.classify(want=("crit_idx",)), case.oracle_classify(oracle)
        assert np.array_equal(got["labels"], ref["labels"]), name
        if kc:
            for idx in np.ndindex(got["labels"].shape[:3]):
                assert np.array_equal(got["crit_idx"][idx], np.nonzero(ref["labels"][idx] == 2)[0]), (name, idx)
        _, lab = case.forward()
        assert np.array_equal(lab.cpu().numpy(), ref["labels"]), name
