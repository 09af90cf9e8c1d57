"""GPU test of the FP64 pair-sum where its waves take no turns (more than one round of workgroups and a C larger than
the L2s): bit for bit the fitness of launches of one round, where they do."""
import pytest
import torch

from paper_1403_4099_amd import pga
from gpu_cases import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant,P", [(0, 1441), (1, 2817)], ids=["8", "16"])   # 23 tiles per 32 or 64 individuals
@pytest.mark.parametrize("N", [2897, 2944])
def test_several_rounds_equal_single_ones(N, variant, P):
    say(f"pair-sum turns N={N} variant={variant}")
    g = torch.Generator(device="cuda").manual_seed(N)
    C = torch.rand(N, N, dtype=torch.float64, device="cuda", generator=g) * 0.2
    C = torch.triu(C, 1)
    C = C + C.T + torch.eye(N, dtype=torch.float64, device="cuda")
    lab = torch.randint(0, 50, (P, N), dtype=torch.int32, device="cuda", generator=g)
    try:
        for p in (P, 704, P - 704, P - 1408):
            pga.tune_set("fp64", N, p, variant)
        got = pga.fitness(C, lab)
        want = torch.cat([pga.fitness(C, x.contiguous()) for x in lab.split(704)])
    finally:
        for p in (P, 704, P - 704, P - 1408):
            pga.tune_set("fp64", N, p, -1)
    assert torch.isfinite(got).all() and torch.equal(got, want)
