"""The states pass (Alg. 1 steps 6-8 per key block) on more blocks than one launch takes: the same states as the heads by
themselves, on both sides of the point where the second launch begins."""
import pytest
import torch

from paper_2605_11354_amd import binding as B

pytestmark = pytest.mark.gpu


def test_states_of_more_than_a_million_blocks():
    H, N = 65535, 17 * 64 - 3                              # 1114095 blocks, launches of 2^20
    g = torch.Generator(device="cuda").manual_seed(5)
    K = torch.randint(0, 0x78, (1, H, N, 64), dtype=torch.uint8, device="cuda", generator=g)
    sK = torch.rand((1, H, 17), device="cuda", generator=g) * 0.02
    hT = torch.full((1, H, 17, B.STATE_ROWS, 64), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.sla_linear_states(B.make_params(1, H, N, 64, 64, 0.1, 0.5, dtype="fp8"), K, K, hT, sK, sK)
    p = B.make_params(1, 2, N, 64, 64, 0.1, 0.5, dtype="fp8")
    edge = (1 << 20) // 17                                 # the head in which the second launch begins
    for h in (0, edge - 1, edge, edge + 1, H - 2):
        one = torch.empty((1, 2, 17, B.STATE_ROWS, 64), dtype=torch.bfloat16, device="cuda")
        k, s = K[:, h:h + 2].clone(), sK[:, h:h + 2].clone()
        B.sla_linear_states(p, k, k, one, s, s)
        torch.cuda.synchronize()
        assert torch.equal(one.view(torch.int16), hT[:, h:h + 2].view(torch.int16)), h
    assert not torch.isnan(hT[0, ::97].float()).any()
