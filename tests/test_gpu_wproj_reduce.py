"""The sum over the partial gradients of W_proj (Alg. 1 step 10) where its form changes: 255 / 256 partials of one matrix
(16 or 64 slices), fewer partials than slices, several batch items per matrix, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2605_11354_amd import binding as B
from paper_2605_11354_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu
GRAD_TOL = 3e-2      # of RMS(dW): phi(Q), O_lin and the states are rounded to bf16 (2^-9 each) on the way; measured 0.7-1.3e-2


# partials of a matrix: B x heads that share it x ceil(ceil(N / 32) / 4), at most 2048 / (4 B H) per head
@pytest.mark.parametrize("Bn,H,N,per_head", [(1, 15, 2170, False), (1, 16, 2048, False), (2, 3, 100, True), (3, 2, 700, True)])
def test_partials_of_the_projection_gradient(oracle, Bn, H, N, per_head):
    cfg = synth.CONFIGS[0].with_(B=Bn, H=H, N=N, proj_per_head=per_head)
    case = G.Case(cfg, k_crit=1, k_neg=0)
    _, lab = case.forward()
    bits = synth.to_bf16_bits(np.random.default_rng(5).standard_normal((Bn, H, N, 64)).astype(np.float32))
    dW = torch.full((H if per_head else 1, 64, 64), float("nan"), dtype=torch.float32, device="cuda")
    B.sla_wproj_grad(case.p, case.Q, G.dev_bf16(bits), dW, case.ws)
    torch.cuda.synchronize()
    d = case.d
    ref = oracle.grad_wproj(case.oracle_params(oracle), d["Q"], d["K"], d["V"], lab.cpu().numpy(),
                            (bits.astype(np.uint32) << 16).view(np.float32).astype(np.float64))
    err = np.abs(dW.cpu().numpy().astype(np.float64) - ref).max()
    assert err <= GRAD_TOL * np.sqrt(np.mean(ref ** 2))
