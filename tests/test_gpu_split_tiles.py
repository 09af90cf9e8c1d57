"""GPU test of MFMA pair-sum launches of at most 512 tiles, which give each column block of a tile a workgroup: the
fitness of their individuals is that of the same individuals in a larger launch, bit for bit, with even and odd numbers
of blocks (the middle block of an odd number has no partner) and a partial last batch."""
import numpy as np
import pytest
import torch

from paper_1403_4099_amd import pga
from gpu_cases import corr, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [0, 1, 2], ids=["8", "4", "16"])     # individuals per workgroup
@pytest.mark.parametrize("N", [20, 65, 128, 129, 333])
def test_split_launch_equals_a_large_one(N, variant):
    say(f"split tiles N={N} variant={variant}")
    C = torch.from_numpy(corr(N, T=200, seed=4)[0].copy()).cuda()
    hi, lo = pga.split(C)
    P = 16 * 513                                             # more than 512 batches of 16
    pop = torch.from_numpy(np.random.default_rng(N).integers(0, max(2, N // 9), size=(P, N)).astype(np.int32)).cuda()
    part = pop[:37].contiguous()
    for p in (P, 37):
        pga.tune_set("bf16x2", N, p, variant)
    try:
        with pga.route(0.0):
            large = pga.fitness(C, pop, "bf16x2", hi=hi, lo=lo)
            small = pga.fitness(C, part, "bf16x2", hi=hi, lo=lo)
    finally:
        for p in (P, 37):
            pga.tune_set("bf16x2", N, p, -1)
    assert torch.equal(small, large[:37])
