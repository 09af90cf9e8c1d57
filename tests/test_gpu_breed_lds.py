"""GPU test of the breed launch that needs the most LDS: 65 536 slots and more, and an instance of the largest N."""
import numpy as np
import pytest
import torch

from paper_1403_4099_amd import pga
from gpu_cases import corr, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sel", ["tournament", "sus"])
def test_the_largest_instance_breeds_beside_65536_slots(sel):
    say(f"breed LDS {sel}")
    N, P = 4096, 9
    rng = np.random.default_rng(5)
    X = rng.standard_normal((N, 64))
    C = np.corrcoef(X)
    np.fill_diagonal(C, 1.0)
    C = torch.from_numpy(np.clip(0.5 * (C + C.T), -1.0, 1.0)).cuda()
    small = torch.from_numpy(corr(8, T=64, seed=1)[0].copy()).cuda()

    def big():
        return pga.make_instance(C, P, stats_rows=3, elites=2, seed=9, instance_id=70, selection=sel)

    alone, beside = big(), big()
    fill = [pga.make_instance(small, 4096, stats_rows=3, elites=2, seed=9, instance_id=k, selection=sel) for k in range(16)]
    pga.Context().evolve([alone], 2, init=True)
    pga.Context().evolve(fill + [beside], 2, init=True)
    assert torch.equal(alone.pop, beside.pop) and torch.equal(alone.fitness, beside.fitness)
    assert torch.equal(alone.stats, beside.stats)
