"""GPU test of evaluations that leave none, one and all of their individuals to the pair-sum and the finish, whose
workgroups end at once in the first case: calls that reuse a workspace, and generations of a captured run."""
import pytest
import torch

from paper_1403_4099_amd import pga
from gpu_cases import corr, say

pytestmark = pytest.mark.gpu

N, P = 200, 96


def _pop(dense, seed=5):
    g = torch.Generator(device="cuda").manual_seed(seed)
    pop = torch.randint(0, N, (P, N), generator=g, device="cuda", dtype=torch.int32)     # about N / 2 pairs
    pop[P - dense:] %= 10                                                               # N^2 / 20 pairs
    return pop


@pytest.mark.parametrize("form", ["fp64", "bf16x2"])
def test_calls_in_one_workspace(form):
    say(f"none, one and all dense, {form}")
    C = torch.from_numpy(corr(N, T=300, seed=2)[0].copy()).cuda()
    hi, lo = pga.split(C)
    ws = torch.full((pga.fitness_ws_bytes(N, P, form),), 0xFF, dtype=torch.uint8, device="cuda")
    for dense in (P, 0, 1, 0, P):
        pop = _pop(dense)
        got = pga.fitness(C, pop, form, hi=hi, lo=lo, ws=ws)
        one = torch.cat([pga.fitness(C, pop[p:p + 1].contiguous(), form, hi=hi, lo=lo) for p in range(P)])
        assert torch.equal(got, one)


@pytest.mark.parametrize("form", ["fp64", "bf16x2"])
@pytest.mark.parametrize("dense", [0, 1, P // 2, P])
def test_generations_of_a_captured_run(form, dense):
    say(f"captured run from {dense} dense, {form}")
    C = torch.from_numpy(corr(N, T=300, seed=2)[0].copy()).cuda()
    hi, lo = pga.split(C)
    runs = []
    for one_by_one in (False, True):
        I = pga.make_instance(C, P, hi=hi, lo=lo, pop=_pop(dense), stats_rows=8, seed=3)
        ctx = pga.Context()
        for g in range(7 if one_by_one else 1):
            I.gen0 = g
            ctx.evolve([I], 1 if one_by_one else 7, form=form)
        assert torch.equal(I.fitness, pga.fitness(C, I.pop, form, hi=hi, lo=lo))
        runs.append(I)
    assert torch.equal(runs[0].pop, runs[1].pop) and torch.equal(runs[0].fitness, runs[1].fitness)
