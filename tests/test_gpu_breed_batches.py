"""GPU test of batches that breed in the shapes of large launches (16 384 and 65 536 slots and more: several slots a
lane group, elites copied by the breed kernel where the ranking is a launch of its own) with SUS, stopping and plain
instances together: every instance equals its own run, whose launch has fewer than 4096 slots."""
import numpy as np
import pytest
import torch

from paper_1403_4099_amd import pga
from gpu_cases import corr, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_inst,P", [(34, 500), (70, 950)], ids=["16k", "64k"])
@pytest.mark.parametrize("stops", [False, True], ids=["fold", "ranked"])
def test_mixed_batches_equal_their_instances_alone(n_inst, P, stops):
    say(f"breed batch {n_inst} x {P} stops={stops}")
    assert n_inst * P >= (65536 if P > 900 else 16384) and P < 4096
    G = 5
    rng = np.random.default_rng(n_inst)
    specs = []                                       # N, selection, stall, elites
    for i in range(n_inst):
        specs.append((int(rng.integers(5, 300)), "sus" if stops and i % 3 == 0 else "tournament",
                      2 if stops and i % 4 == 1 else 0, (2, 0, 33)[i % 3]))
    Cs = [torch.from_numpy(corr(N, T=64, seed=300 + i)[0].copy()).cuda() for i, (N, *_r) in enumerate(specs)]

    def inst(i):
        _, sel, stall, E = specs[i]
        I = pga.make_instance(Cs[i], P, stats_rows=G + 1, elites=E, seed=41, instance_id=i, selection=sel, stall_gens=stall,
                              tol=1e9)
        I.stats.fill_(float("nan"))
        return I

    batch = [inst(i) for i in range(n_inst)]
    pga.Context().evolve(batch, G, init=True)
    torch.cuda.synchronize()
    for i, b in enumerate(batch):
        a = inst(i)
        pga.Context().evolve([a], G, init=True)
        assert torch.equal(a.pop, b.pop) and torch.equal(a.fitness, b.fitness), (i, specs[i])
        assert torch.equal(torch.nan_to_num(a.stats, nan=7.0), torch.nan_to_num(b.stats, nan=7.0)), (i, specs[i])
        assert a.term_state() == b.term_state(), (i, specs[i])
    assert any(b.term_state()["stopped"] for b in batch) == stops
