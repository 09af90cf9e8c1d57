"""GPU test of launches with more pair-sum tiles than a list is made for (16384): their fitness is that of the same
individuals in small launches, bit for bit, where few, many and all of them are left to the pair-sum."""
import numpy as np
import pytest
import torch

from paper_1403_4099_amd import pga
from gpu_cases import corr, say

pytestmark = pytest.mark.gpu

N, P = {"bf16x2": 200, "fp64": 1000}, {"bf16x2": 66001, "fp64": 66001}   # ceil(P / 8) 2 and ceil(P / 32) 8 tiles


def _pop(form, dense):
    """Random labels (about N / 2 pairs), and on a share of the individuals ten clusters (N^2 / 20 pairs)."""
    g = torch.Generator(device="cuda").manual_seed(7)
    n, p = N[form], P[form]
    pop = torch.randint(0, n, (p, n), generator=g, device="cuda", dtype=torch.int32)
    if dense:
        rows = torch.arange(p, device="cuda") % dense == dense // 2
        pop[rows] %= 10
    return pop


def _chunks(C, pop, form, hi, lo):
    return torch.cat([pga.fitness(C, c.contiguous(), form, hi=hi, lo=lo) for c in pop.split(12000)])


@pytest.mark.parametrize("form", ["bf16x2", "fp64"])
@pytest.mark.parametrize("dense", [0, 5003, 3, 1], ids=["none", "few", "third", "all"])
def test_listed_tiles_give_the_fitness_of_small_launches(form, dense):
    say(f"tile lists {form} every {dense}")
    C = torch.from_numpy(corr(N[form], T=300, seed=2)[0].copy()).cuda()
    hi, lo = pga.split(C)
    pop = _pop(form, dense)
    want = _chunks(C, pop, form, hi, lo)
    assert torch.equal(pga.fitness(C, pop, form, hi=hi, lo=lo), want)
    if dense:
        with pga.route(1.0 / 32.0):                           # another share of them
            got = pga.fitness(C, pop, form, hi=hi, lo=lo)
            assert torch.equal(got, _chunks(C, pop, form, hi, lo))


def test_listed_tiles_in_a_captured_run():
    """Generations of one captured run reuse the lists in turn; replayed, it gives the same."""
    say("tile lists captured")
    C = torch.from_numpy(corr(N["bf16x2"], T=300, seed=2)[0].copy()).cuda()
    hi, lo = pga.split(C)
    pop = _pop("bf16x2", 3)
    runs = []
    ctx = pga.Context()
    for eager in (True, False, False):
        I = pga.make_instance(C, P["bf16x2"], hi=hi, lo=lo, pop=pop.clone(), stats_rows=6, seed=3)
        if runs:
            I.pop, I.pop_tmp, I.fitness = runs[-1][2:]         # the same buffers: the same captured graph
            I.pop.copy_(pop)
        ctx.evolve([I], 5, form="bf16x2", eager=eager)
        torch.cuda.synchronize()
        assert torch.equal(I.fitness, _chunks(C, I.pop, "bf16x2", hi, lo))
        runs.append((I.pop.clone(), I.fitness.clone(), I.pop, I.pop_tmp, I.fitness))
    for r in runs[1:]:
        assert torch.equal(r[0], runs[0][0]) and torch.equal(r[1], runs[0][1])
    assert ctx.graphs() == 1
