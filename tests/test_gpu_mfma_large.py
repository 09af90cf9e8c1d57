"""GPU test of MFMA pair-sum launches at the largest N with many tiles (two workgroups per CU; from 16384 tiles also
listed): bit for bit the fitness of smaller launches."""
import pytest
import torch

from paper_1403_4099_amd import pga
from gpu_cases import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,P", [(4033, 2049), (4096, 2050), (4096, 4105)])      # 257, 257 and 514 batches of 32 tiles
def test_many_tiles_equal_few(N, P):
    say(f"MFMA many tiles N={N} P={P}")
    g = torch.Generator(device="cuda").manual_seed(N + P)
    C = torch.rand(N, N, dtype=torch.float64, device="cuda", generator=g) * 0.2
    C = torch.triu(C, 1)
    C = C + C.T + torch.eye(N, dtype=torch.float64, device="cuda")
    hi, lo = pga.split(C)
    lab = torch.randint(0, 60, (P, N), dtype=torch.int32, device="cuda", generator=g)
    got = pga.fitness(C, lab, "bf16x2", hi=hi, lo=lo)
    want = torch.cat([pga.fitness(C, x.contiguous(), "bf16x2", hi=hi, lo=lo) for x in lab.split(1000)])
    assert torch.isfinite(got).all() and torch.equal(got, want)
