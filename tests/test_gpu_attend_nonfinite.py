"""Infinities and NaN in Q or K stay in the rows whose softmax they reach: every other row of the attention kernel (Alg. 1
steps 4-5) is that of the oracle, on lists of a few entries and of more than one window, in every form of the kernel, and
on the short-list kernel."""
import numpy as np
import pytest
import torch

from paper_2605_11354_amd import binding as B
from paper_2605_11354_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu
INF, NAN = 0x7F80, 0x7FC0                                  # bf16 (with 0x8000: the negative)


def _case(bq, dtype, nkb, length, seed):
    cfg = synth.CONFIGS[1].with_(H=1, N=nkb * 64 - 9, bq=bq)
    d = {n: a.copy() if isinstance(a, np.ndarray) else a for n, a in synth.make_inputs(cfg).items()}
    if dtype == "fp8":
        cfg = cfg.with_(dtype="fp8")
        for t, blk in (("Q", bq), ("K", 64), ("V", 64)):
            d[t], d["s" + t] = synth.quantise_e4m3_blocks(d[t], blk)
    rng = np.random.default_rng(seed)
    Nqb = -(-cfg.N // bq)
    lab = np.ones((1, 1, Nqb, nkb), np.int8)
    for i in range(Nqb):
        lab[0, 0, i, rng.choice(nkb, length, replace=False)] = 2
    return cfg, d, lab


def _run(cfg, d, lab, length, launch=0):
    case = G.Case(cfg, d, k_crit=length, k_neg=0)
    sparse = G.sparse_f32(case, lab, launch)
    labd = torch.from_numpy(lab).cuda()
    whole = torch.full((1, 1, cfg.N, 64), 7.0, dtype=torch.bfloat16, device="cuda")
    B.sla_forward_with_labels(case.p, case.Q, case.K, case.V, case.W, labd, whole, case.sQ, case.sK, case.sV, case.ws)
    torch.cuda.synchronize()
    return case, sparse, G.bf16_tensor_to_f64(whole)[0, 0]


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("bq,length,launch", [(64, 2, 0), (64, 3, 0), (64, 9, 0), (64, 34, 0), (64, 68, 0), (128, 3, 0), (128, 9, 0), (128, 34, 0), (128, 68, 0),
                                              (128, 3, 769), (128, 9, 769), (128, 68, 769)])
def test_query_rows_with_infinities_and_nan(oracle, bq, length, launch, dtype):
    cfg, d, lab = _case(bq, dtype, 70, length, length)
    case, _, _ = _run(cfg, d, lab, length)
    ref = case.oracle_attend(oracle, lab, want_parts=True)
    rows = {3: NAN, 64 + 17: INF, 128 + 40: 0x8000 | NAN, 5 * 128 + 31: INF, cfg.N - 1: NAN}
    for r, bits in rows.items():
        if dtype == "bf16":
            d["Q"][0, 0, r, r % 64] = bits
        else:
            d["Q"][0, 0, r, r % 64] = 0x7F                  # E4M3 has no infinities: NaN
    huge = [300, 301, 450, 1000, 1001, 2222]                # and finite rows whose logits leave the resolution of fp32: anything, but alone
    if dtype == "bf16":
        for r, size in zip(huge, [1e30, -1e30, 3e38, -1e12, 3e9, 1e20]):
            d["Q"][0, 0, r, :7 * (r % 2) + 1] = np.float32(size).view(np.uint32) >> 16
    _, sparse, whole = _run(cfg, d, lab, length, launch)
    good = np.ones(cfg.N, bool)
    good[list(rows)] = False
    assert np.isnan(sparse[~good]).all() and np.isnan(whole[~good]).all()
    good[huge] = dtype != "bf16"
    full = lambda part: part.reshape(-1, 64)[:cfg.N]
    for got, part in ((sparse, "O_sparse"), (whole, "O")):
        want = full(ref[part])
        strict, err = G.output_error(got[good], want[good])
        print(f"bq={bq} {dtype} {length} {part}: {strict:.3e}, {err:.3e} beyond a bf16 store")
        assert (strict if part == "O_sparse" else err) <= G.TOL[dtype]


@pytest.mark.parametrize("bq,dtype,launch", G.ATTEND_FORMS)
def test_a_nan_row_in_every_group_of_rows(oracle, bq, dtype, launch):
    """One query in sixteen is NaN, so that no wave has a group of rows without one."""
    cfg, d, lab = _case(bq, dtype, 20, 9, 5)
    case, _, _ = _run(cfg, d, lab, 9)
    want = case.oracle_attend(oracle, lab, want_parts=True)["O_sparse"].reshape(-1, 64)[:cfg.N]
    d["Q"][0, 0, 3::16, 7] = NAN if dtype == "bf16" else 0x7F
    _, sparse, _ = _run(cfg, d, lab, 9, launch)
    bad = np.arange(cfg.N) % 16 == 3
    assert np.isnan(sparse[bad]).all()
    err, _ = G.output_error(sparse[~bad], want[~bad])
    print(f"bq={bq} {dtype} {launch}: {err:.3e}")
    assert err <= G.TOL[dtype]


@pytest.mark.parametrize("bq,launch", [(64, 0), (128, 0), (128, 769)])
@pytest.mark.parametrize("length", [2, 9, 68])
def test_keys_with_an_infinity(bq, launch, length):
    """K[t][c] = +inf: rows with q[c] > 0 that attend to t see a logit of +inf (NaN out), rows with q[c] < 0 one of -inf (weight
    0), rows with q[c] = 0 NaN."""
    cfg, d, lab = _case(bq, "bf16", 70, length, 100 + length)
    keys = {(11, 5), (37 * 64 + 50, 20)}
    for t, c in keys:
        d["K"][0, 0, t, c] = INF
        lab[0, 0, :, t // 64] = np.where(np.arange(lab.shape[2]) % 3 == 0, lab[0, 0, :, t // 64], 1)      # one row in three at most attends to it
    lab[0, 0, ::5, 0], lab[0, 0, ::5, 1:] = 2, np.where(np.cumsum(lab[0, 0, ::5, 1:] == 2, axis=1) < length, lab[0, 0, ::5, 1:], 1)
    _, sparse, _ = _run(cfg, d, lab, length, launch)
    f = lambda b: (b.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    q, k, v = f(d["Q"][0, 0]), f(d["K"][0, 0]), f(d["V"][0, 0])
    want = np.zeros((cfg.N, 64))
    with np.errstate(invalid="ignore"):
        for i in range(lab.shape[2]):
            js = np.flatnonzero(lab[0, 0, i] == 2)[:length]
            t = np.concatenate([np.arange(64 * j, min(64 * j + 64, cfg.N)) for j in js]) if len(js) else np.zeros(0, int)
            if len(t) == 0:
                continue
            qi, kt = q[i * bq:(i + 1) * bq], k[t]
            s = (qi[:, None, :] * kt[None]).sum(-1) * 0.125        # the products themselves: 0 inf = NaN
            w = np.exp(s - s.max(axis=1, keepdims=True))
            want[i * bq:i * bq + len(qi)] = (w @ v[t]) / w.sum(axis=1, keepdims=True)
    bad = np.isnan(want).any(axis=1)
    assert 0 < bad.sum() < cfg.N // 2
    assert np.array_equal(np.isnan(sparse), np.isnan(want))
    err = np.abs(sparse[~bad] - want[~bad]).max() / np.sqrt(np.mean(want[~bad] ** 2))
    print(f"bq={bq} {length}: {err:.3e}, {bad.sum()} rows NaN")
    assert err <= G.TOL["bf16"]
