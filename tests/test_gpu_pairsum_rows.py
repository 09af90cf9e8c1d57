"""GPU test of the FP64 pair-sum's row walk: last chunks that reach past N, the smallest N, populations that do
not fill the last wave, in both group sizes, against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1403_4099_amd import pga
from gpu_cases import corr, fitness_tol, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [0, 1], ids=["8", "16"])     # individuals per wave
@pytest.mark.parametrize("N,P", [(1, 1), (3, 9), (63, 33), (65, 31), (127, 65), (131, 8), (200, 70)])
def test_rows_at_the_edges_of_a_chunk(N, P, variant):
    say(f"pair-sum rows N={N} P={P} variant={variant}")
    C, _ = corr(N, T=96, seed=N)
    lab = np.random.default_rng(N + P).integers(0, max(1, N // 9), size=(P, N)).astype(np.int32)
    pga.tune_set("fp64", N, P, variant)
    try:
        with pga.route(0.0):
            got = pga.fitness(torch.from_numpy(C.copy()).cuda(), torch.from_numpy(lab).cuda()).cpu().numpy()
    finally:
        pga.tune_set("fp64", N, P, -1)
    want, mag = O.fitness(C, lab, want_mag=True)
    ok = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), ok)
    assert np.all(np.abs(got[ok] - want[ok]) <= fitness_tol(mag)[ok])


@pytest.mark.parametrize("variant", [0, 1], ids=["8", "16"])
@pytest.mark.parametrize("N", [1000, 961, 65])
def test_the_matrix_may_end_its_memory(N, variant):
    """The last rows of a chunk that reaches past N: the result is that of a matrix with NaN behind it, and no load
    needs what is there (the walk takes row N - 1 instead)."""
    say(f"pair-sum at the end of C, N={N} variant={variant}")
    C, _ = corr(N, T=96, seed=1)
    lab = torch.from_numpy(np.random.default_rng(N).integers(0, 9, size=(40, N)).astype(np.int32)).cuda()
    tail = torch.full((N + 80, N), float("nan"), dtype=torch.float64, device="cuda")
    tail[:N] = torch.from_numpy(C.copy()).cuda()
    pga.tune_set("fp64", N, 40, variant)
    try:
        with pga.route(0.0):
            a, b = pga.fitness(tail[:N].clone(), lab), pga.fitness(tail[:N], lab)
    finally:
        pga.tune_set("fp64", N, 40, -1)
    assert torch.isfinite(a).any() and torch.equal(a, b)
