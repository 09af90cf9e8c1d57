"""GPU test of the rank kernel of launches that select by SUS (a sort by one workgroup per instance, P <= 4096) and of
the general kernels above it: P at the edges of waves, of the padded sort and of the three kernels, populations with
many equal fitness values and invalid individuals. The next population is compared bit for bit with the oracle's
breeding, the statistics row with the fitness."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1403_4099_amd import pga
from gpu_cases import corr, say

pytestmark = pytest.mark.gpu

SIZES = [(2, 0), (2, 1), (3, 2), (63, 2), (64, 2), (65, 10), (128, 0), (1000, 10), (1023, 2), (1024, 32), (1025, 2),
         (2048, 2), (2049, 1), (3500, 10), (4096, 2), (4097, 2)]


@pytest.mark.parametrize("P,E", SIZES)
@pytest.mark.parametrize("bad", ["none", "some", "all"])
def test_ranks_weights_and_pointers(P, E, bad):
    say(f"SUS sorted P={P} E={E} bad={bad}")
    N = 5                                                    # 52 partitions: nearly every fitness has equals
    C, _ = corr(N, T=64, seed=3)
    rng = np.random.default_rng(P)
    pop = rng.integers(0, N, size=(P, N)).astype(np.int32)
    if bad != "none":
        pop[rng.random(P) < (0.4 if bad == "some" else 2.0), 0] = N    # out of range: fitness -inf
    I = pga.make_instance(torch.from_numpy(C.copy()).cuda(), P, pop=torch.from_numpy(pop).cuda(), stats_rows=2,
                          elites=E, seed=5, instance_id=2, selection="sus")
    f = pga.fitness(I.C, I.pop).cpu().numpy()
    pga.Context().evolve([I], 1)
    want = O.breed(pop, f, E=E, seed=5, inst=2, gen=0, selection=1)
    assert np.array_equal(I.pop.cpu().numpy(), want)
    best, mean, ninv, at = I.stats[0].cpu().numpy()
    fin = np.isfinite(f)
    order = np.lexsort((np.arange(P), -f))
    assert (best, ninv, at) == (f[order[0]], P - fin.sum(), order[0])
    assert mean == (-np.inf if not fin.any() else pytest.approx(f[fin].mean(), rel=1e-12, abs=1e-300))
