"""GPU tests of the cluster-pair kernel's lane groups: 16 lanes per individual (N <= 32), 32 (N <= 64), a
wave (N <= 512), a workgroup (N <= 2048), at the edges of each, with populations whose last workgroup is
partly empty; and of the small instances' own handling of C entries outside [-1, 1]."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1403_4099_amd import pga, synth
from gpu_cases import corr, fitness_tol, say

pytestmark = pytest.mark.gpu


def _g(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


EDGES = [(1, 3), (2, 17), (16, 15), (17, 33), (32, 16), (33, 9), (64, 8), (65, 5), (512, 6), (513, 3), (2047, 2),
         (2048, 2)]


@pytest.mark.parametrize("N,P", EDGES, ids=[f"N{n}-P{p}" for n, p in EDGES])
def test_every_group_size_matches_the_oracle(N, P):
    """One cluster, a few large ones, pairs, and singletons, every pair on the route: the chains' longest and
    shortest forms. Fixed-point sums and FP64 logs: 1e-10 of the log terms' magnitude."""
    say(f"eval groups N={N} P={P}")
    C, _ = corr(N, T=64, seed=N)
    rng = np.random.default_rng(N)
    pop = np.stack([rng.integers(0, max(1, K), size=N) for K in
                    [(1, 2, max(1, N // 8), max(1, N // 2), N)[i % 5] for i in range(P)]]).astype(np.int32)
    pop[-1] = rng.permutation(N)                      # all singletons
    with pga.route(1.0):
        f, ns, cs = pga.fitness(_g(C), _g(pop), "fp64", want_ns=True, want_cs=True)
    f_o, ns_o, cs_o, mag = O.fitness(C, pop, want_ns=True, want_cs=True, want_mag=True)
    assert np.array_equal(ns.cpu().numpy(), ns_o)
    assert np.all(np.abs(cs.cpu().numpy() - cs_o) <= 1e-12 * np.maximum(1.0, ns_o.astype(float) ** 2))
    assert np.all(np.abs(f.cpu().numpy() - f_o) <= fitness_tol(mag, 1e-10))
    assert f.cpu().numpy()[-1] == 0.0


@pytest.mark.parametrize("form", ["fp64", "bf16x2"])
@pytest.mark.parametrize("N", [3, 16, 17, 31, 33, 63, 64])
def test_small_instances_with_entries_out_of_range_equal_the_pair_sum_route(N, form):
    """N <= 64 has no pair-sum launch behind it: an individual whose clusters meet an entry above 1 (or a NaN,
    or a diagonal above 1) is evaluated in the kernel, with the pair-sum's bits, n_s, c_s and status, in
    groups that share a wave with ordinary and with invalid individuals."""
    say(f"small out of range N={N} {form}")
    C, _ = corr(N, T=64, seed=300 + N)
    C = C.copy()
    a, b = 1, N - 1
    C[a, b] = C[b, a] = 1.5
    P = 37
    pop = synth.random_labelings(P, N, seed=N, K=max(2, N // 3))
    bad = np.zeros(P, dtype=bool)
    for p in range(P):
        if p % 4 == 1:
            pop[p, a] = pop[p, b]
        bad[p] = pop[p, a] == pop[p, b]
    invalid = np.arange(P) % 9 == 5
    pop[invalid, 0] = N
    sel = bad & ~invalid
    assert sel.sum() > 3

    def run(Cm, labels, frac):
        Cg = _g(Cm)
        hi, lo = pga.split(Cg) if form == "bf16x2" else (None, None)
        st = pga.new_status()
        with pga.route(frac):
            out = pga.fitness(Cg, _g(labels), form, hi=hi, lo=lo, want_ns=True, want_cs=True, status=st)
        return [x.cpu().numpy() for x in out] + [st.cpu().numpy()]

    got, want = run(C, pop, 1.0 / 64), run(C, pop, 0.0)
    for x, y in zip(got[:3], want[:3]):
        assert np.array_equal(x[sel], y[sel])
        assert np.array_equal(x[invalid], y[invalid])
    assert np.all(np.isneginf(got[0][invalid])) and got[3][0] == int(invalid.sum())
    # only the individuals that meet the entry, in both routes: the status words too
    got, want = run(C, pop[sel], 1.0 / 64), run(C, pop[sel], 0.0)
    for x, y in zip(got, want):
        assert np.array_equal(x, y)
    for i, j, v in ((a, b, np.nan), (b, b, 1.25)):
        D = C.copy()
        D[i, j] = D[j, i] = v
        got, want = run(D, pop[sel], 1.0 / 64), run(D, pop[sel], 0.0)
        for x, y in zip(got, want):
            assert np.array_equal(x, y)
