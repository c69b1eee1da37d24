"""Rows of 65 to 256 key blocks, where the classifier keeps two to four logits per lane and takes both ranks in one descent: the
first and last length of each form, ragged ends, query blocks past the end, ranks next to each other, at the ends and equal, ties;
block means, logits, labels and lists bit for bit against the oracle."""
import numpy as np
import pytest

from paper_2605_11354_amd import synth
from tests import gpu_util as G
from tests.test_gpu_short_rows import _check, _variants

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nkb,short,bq,dtype", [(65, 63, 64, "bf16"), (128, 0, 128, "fp8"), (129, 30, 128, "bf16"), (192, 1, 64, "fp8"),
                                                (193, 63, 128, "fp8"), (256, 0, 128, "bf16")])
def test_fused_rows_at_their_edges(oracle, nkb, short, bq, dtype):
    cfg = synth.CONFIGS[4 if dtype == "fp8" else 0].with_(B=1, H=2, N=nkb * 64 - short, bq=bq, crit_frac=0.06, neg_frac=0.5, n_clusters=8)
    _check(oracle, G.Case(cfg), (nkb, short, bq, dtype))


@pytest.mark.parametrize("nkb,kc,kn", [(65, 1, 64), (100, 50, 49), (128, 0, 128), (130, 130, 0), (172, 9, 0), (200, 0, 5), (256, 255, 1)])
def test_fused_rows_with_ties_and_extreme_counts(oracle, nkb, kc, kn):
    cfg = synth.CONFIGS[0].with_(H=1, N=nkb * 64 - 17, bq=128, n_clusters=16)
    for name, dd in _variants(cfg, synth.make_inputs(cfg)):
        case = G.Case(cfg, dd, k_crit=kc, k_neg=kn)
        got, ref = case.classify(want=("crit_idx",)), case.oracle_classify(oracle)
        assert np.array_equal(got["labels"], ref["labels"]), (nkb, kc, kn, name)
        if kc:
            for idx in np.ndindex(got["labels"].shape[:3]):
                assert np.array_equal(got["crit_idx"][idx], np.nonzero(ref["labels"][idx] == 2)[0]), (nkb, name, idx)
