"""GPU test of the reuse of captured graphs by later mixes of instances: mixes whose totals of tiles and individuals and
whose largest N round to the same values share a graph where the evaluation's and the breeding's workgroups and
LDS differ within one value of theirs, and every replay gives the populations of an eager run."""
import pytest
import torch

from paper_1403_4099_amd import pga
from gpu_cases import corr, say

pytestmark = pytest.mark.gpu

MIXES = {
    "lds": [(290,), (300,), (310,), (320,)],                   # one number of workgroups per CU
    "evaluation": [(300, 20), (300, 40), (300, 32)],           # 16 and 8 individuals a workgroup beside 4
    "both": [(300, 20, 20), (310, 33, 64), (290, 20, 50)],
}


@pytest.mark.parametrize("form", ["fp64", "bf16x2"])
@pytest.mark.parametrize("name", MIXES)
def test_mixes_of_one_shape_share_a_graph(name, form):
    say(f"graph reuse {name} {form}")
    P, G = 64, 3
    ctx = pga.Context()
    ctx.ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")     # one workspace for every mix
    for rep in range(2):
        for mix in MIXES[name]:
            runs = []
            for eager in (True, False):
                insts = []
                for k, N in enumerate(mix):
                    C = torch.from_numpy(corr(N, T=64, seed=N)[0].copy()).cuda()
                    hi, lo = pga.split(C) if form == "bf16x2" else (None, None)
                    insts.append(pga.make_instance(C, P, hi=hi, lo=lo, stats_rows=G + 1, elites=2, seed=3 + rep, instance_id=k))
                (pga.Context() if eager else ctx).evolve(insts, G, form=form, init=True, eager=eager)
                torch.cuda.synchronize()
                runs.append(insts)
            for a, b in zip(*runs):
                assert torch.equal(a.pop, b.pop) and torch.equal(a.fitness, b.fitness) and torch.equal(a.stats, b.stats)
    assert ctx.graphs() == 1
