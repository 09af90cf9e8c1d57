"""GPU test of listed pair-sum tiles (more than 16384 of them) over ragged batches: instances without tiles (N <= 64),
above the cluster-pair kernel's N (2048), stopped before the call and stopped by it, in every tile order and
group size. Every instance has the bits of its own run, which is too small for a list."""
import numpy as np
import pytest
import torch

from paper_1403_4099_amd import pga
from gpu_cases import corr, say

pytestmark = pytest.mark.gpu

G = 3
# N, P (times the case's factor), how the instance stops
MFMA = [(200, 20000, ""), (40, 500, ""), (300, 20000, ""), (150, 9000, "before"), (2100, 300, ""), (64, 100, "during"),
        (260, 10000, "during"), (1000, 700, "")]
FP64 = [(500, 30000, ""), (40, 500, ""), (150, 60000, "before"), (2100, 1000, ""), (64, 100, "during"),
        (450, 30000, "during"), (1000, 9000, ""), (300, 40000, "")]


def _fold(n):
    return ((n + 63) // 64 + 1) // 2


def _pop(N, P, seed):
    """Random labels, and ten clusters on every third individual and on a run of a hundred."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    pop = torch.randint(0, N, (P, N), generator=g, device="cuda", dtype=torch.int32)
    pop[::3] %= 10
    pop[P // 2:P // 2 + 100] %= 10
    return pop


@pytest.mark.parametrize("form,variant,times", [("bf16x2", 0, 1), ("bf16x2", 1, 1), ("bf16x2", 2, 2), ("bf16x2", 3, 1),
                                                ("bf16x2", 5, 1), ("fp64", 0, 1), ("fp64", 1, 2), ("fp64", 2, 1),
                                                ("fp64", 4, 1)])
def test_ragged_batches_equal_their_instances_alone(form, variant, times):
    specs = [(N, P * times, how) for N, P, how in (MFMA if form == "bf16x2" else FP64)]
    ipg, order, kind = pga.variants(form)[variant]
    assert kind == 0
    per = 4 * ipg if form == "fp64" else ipg
    tiles = sum(_fold(N) * -(-P // per) for N, P, _ in specs if N > 64)
    say(f"tile list batch {form} group {ipg} order {order}: {tiles} tiles")
    assert tiles > 16384
    Cs = [torch.from_numpy(corr(N, T=64, seed=N)[0].copy()).cuda() for N, _, _ in specs]

    def inst(k):
        N, P, how = specs[k]
        hi, lo = pga.split(Cs[k]) if form == "bf16x2" else (None, None)
        I = pga.make_instance(Cs[k], P, hi=hi, lo=lo, pop=_pop(N, P, k), stats_rows=G + 1, elites=2, seed=5, instance_id=k,
                              stall_gens=1 if how else 0, tol=1e9)
        I.stats.fill_(float("nan"))
        if how == "before":
            pga.Context().evolve([I], 2, form=form)
            assert I.term_state()["stopped"] == 1
        return I

    batch = [inst(k) for k in range(len(specs))]
    big_n, total = 2560, sum(P for _, P, _ in specs)               # the launch's rounded largest N: the table's key
    pga.tune_set(form, big_n, total, variant)
    try:
        pga.Context().evolve(batch, G, form=form)
        torch.cuda.synchronize()
    finally:
        pga.tune_set(form, big_n, total, -1)
    for k, b in enumerate(batch):
        a = inst(k)
        pga.Context().evolve([a], G, form=form)
        assert torch.equal(a.pop, b.pop) and torch.equal(a.fitness, b.fitness), specs[k]
        assert torch.equal(torch.nan_to_num(a.stats, nan=7.0), torch.nan_to_num(b.stats, nan=7.0)), specs[k]
        assert a.term_state() == b.term_state(), specs[k]
        assert a.term_state()["stopped"] == (1 if specs[k][2] else 0)
