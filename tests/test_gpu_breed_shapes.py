"""GPU tests of the breed launch's shapes: lanes per slot and slots per workgroup depend on the launch's size
and each instance's N, the children do not. Populations are compared bit for bit with the oracle's breeding
and between a small launch and large ones that hold the same instance."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1403_4099_amd import pga
from gpu_cases import corr, say

pytestmark = pytest.mark.gpu


def _g(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _inst(C, P, k, sel, **kw):
    return pga.make_instance(_g(C), P, stats_rows=3, elites=kw.pop("E", 2), seed=77, instance_id=k, selection=sel, **kw)


# 16 lanes per slot and more, whole and partial passes, odd N, crossover words of one and several draws
@pytest.mark.parametrize("N,P,E,sel", [(2, 5, 1, "tournament"), (31, 40, 0, "tournament"), (33, 70, 3, "sus"),
                                       (64, 33, 2, "tournament"), (129, 41, 5, "tournament"), (257, 30, 2, "sus"),
                                       (1025, 9, 2, "tournament"), (2050, 5, 1, "tournament")])
def test_children_match_the_oracle_at_every_split(N, P, E, sel):
    say(f"breed split N={N} P={P} {sel}")
    C, _ = corr(N, T=64, seed=N)
    ctx = pga.Context()
    I = _inst(C, P, 3, sel, E=E)
    ctx.evolve([I], 0, init=True)
    pop, f = I.pop.cpu().numpy(), I.fitness.cpu().numpy()
    ctx.evolve([I], 1)
    nxt = O.breed(pop, f, E=E, seed=77, inst=3, gen=0, selection=pga.SELECTIONS[sel])
    assert np.array_equal(I.pop.cpu().numpy(), nxt)


@pytest.mark.parametrize("fill", [4500, 17000, 66000], ids=["4k", "16k", "64k"])
def test_an_instance_breeds_the_same_in_launches_of_every_size(fill):
    """The instance under test beside a filler of `fill` slots (N = 9): the shapes of launches of 4096, 16 384
    and 65 536 slots and more."""
    say(f"breed beside {fill} slots")
    Cf, _ = corr(9, T=64, seed=1)
    for N, sel in ((300, "tournament"), (75, "sus")):
        C, _ = corr(N, T=64, seed=N)
        alone, beside = _inst(C, 50, 1, sel), _inst(C, 50, 1, sel)
        filler = _inst(Cf, fill, 2, "tournament")
        pga.Context().evolve([alone], 2, init=True)
        pga.Context().evolve([filler, beside], 2, init=True)
        assert torch.equal(alone.pop, beside.pop) and torch.equal(alone.fitness, beside.fitness)
        assert torch.equal(alone.stats, beside.stats)


@pytest.mark.parametrize("fill", [0, 4500], ids=["alone", "4k"])
def test_a_stopped_instance_stays_as_it_is_without_a_stop_test(fill):
    """Stopped by the termination test after an odd number of generations, then evolved by a call without
    the test, whose breed launch does the ranking."""
    say(f"stopped instance, then no stop test, beside {fill} slots")
    C, _ = corr(40, T=64, seed=4)
    Cf, _ = corr(9, T=64, seed=1)
    ctx = pga.Context()
    I = _inst(C, 50, 1, "tournament", stall_gens=1, tol=1e9)
    ctx.evolve([I], 2, init=True)
    st = I.term_state()
    assert st["stopped"] == 1 and st["call_gens"] == 1
    I.stall_gens = 0
    before = [x.clone() for x in (I.pop, I.fitness, I.stats)]
    others = [_inst(Cf, fill, 2, "tournament")] if fill else []
    ctx.evolve(others + [I], 2, init=False)
    for x, b in zip((I.pop, I.fitness, I.stats), before):
        assert torch.equal(torch.nan_to_num(x.double(), nan=7.0), torch.nan_to_num(b.double(), nan=7.0))
    assert I.term_state() == dict(st, call_gens=0)
