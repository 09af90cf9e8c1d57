"""GPU test of the rule that chooses the correlation's launch form, on both sides of its lines: C against FP64 on the
host, and the same bits whether the split is asked for or not.

Tolerance, as derived for the forms themselves: any summation order of a Gram entry over its norm is within
(T + 8) 2^-53 of the exact value, 1e-12 at these T."""
import numpy as np
import pytest
import torch

from paper_1403_4099_amd import pga
from gpu_cases import say

pytestmark = pytest.mark.gpu

SIZES = [(480, 1024), (480, 1025), (481, 768), (496, 1024), (608, 768), (608, 769), (609, 256), (704, 257), (705, 64)]


@pytest.mark.parametrize("N,T", SIZES, ids=[f"N{n}-T{t}" for n, t in SIZES])
def test_both_sides_of_the_form_rule(N, T):
    say(f"corr rule N={N} T={T}")
    rng = np.random.default_rng(N + T)
    R = 0.5 * rng.standard_normal(T)[None, :] + rng.standard_normal((N, T))
    Rg = torch.from_numpy(R).cuda()
    C, hi, lo = pga.correlate(Rg, split=True)
    assert torch.equal(C, pga.correlate(Rg, split=False))
    hi2, lo2 = pga.split(C)
    assert torch.equal(hi, hi2) and torch.equal(lo, lo2)
    X = R - R.mean(axis=1, keepdims=True)
    s = np.sqrt((X * X).sum(axis=1))
    E = X @ X.T / np.outer(s, s)
    np.fill_diagonal(E, 1.0)
    assert np.max(np.abs(C.cpu().numpy() - E)) <= 1e-12
