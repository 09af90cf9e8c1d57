"""GPU tests of the Gram kernel's slices and last chunks: tile counts on both sides of a change in the number
of slices (36 to 66 tiles: 7, 5, 4 and 3 slices; 136 and above: one), sample counts whose slices end after
1, 2, 3 or 4 quarters of a 32-sample chunk, in the middle of a quarter, or short of the others.

Tolerance, derived before the first run: a Gram entry over its norm is a sum of T products of total absolute
size at most 1 (Cauchy-Schwarz), so any summation order is within (T + 8) 2^-53 of the exact value (8: means,
norms, division) on both sides: 1e-12 at T <= 4200."""
import numpy as np
import pytest
import torch

from paper_1403_4099_amd import pga
from gpu_cases import say

pytestmark = pytest.mark.gpu

SIZES = [(1024, 7 * 64 + 1), (1025, 5 * 72), (1026, 5 * 88 - 3), (1153, 4 * 80 - 25), (1281, 3 * 96 + 9), (1307, 295),
         (1925, 41), (705, 2), (705, 31), (706, 33), (800, 64 * 9 + 5), (353, 1037)]


@pytest.mark.parametrize("N,T", SIZES, ids=[f"N{n}-T{t}" for n, t in SIZES])
def test_gram_slices_and_last_chunks(N, T):
    say(f"gram slices N={N} T={T}")
    rng = np.random.default_rng(N * 10007 + T)
    R = 0.5 * rng.standard_normal(T)[None, :] + rng.standard_normal((N, T))
    wide = torch.full((N, T + 3), float("nan"), dtype=torch.float64, device="cuda")   # nothing past T counts
    wide[:, :T] = torch.from_numpy(R)
    C, _, _ = pga.correlate(wide[:, :T], split=True)
    Cg = C.cpu().numpy()
    X = R - R.mean(axis=1, keepdims=True)
    s = np.sqrt((X * X).sum(axis=1))
    E = np.clip((X @ X.T) / np.outer(s, s), -1.0, 1.0)
    np.fill_diagonal(E, 1.0)
    assert np.max(np.abs(Cg - E)) <= 1e-12
    assert np.array_equal(Cg, Cg.T) and np.all(np.diag(Cg) == 1.0)

    S0 = X @ X.T / T + np.eye(N)
    S = torch.from_numpy(S0.copy()).cuda()
    pga.ewma(wide[:, :T], S, 0.97)
    W = 0.03 * 0.97 ** np.arange(T - 1, -1, -1.0)
    Y = R - R.mean(axis=0, keepdims=True)
    S_e = 0.97 ** T * S0 + (Y * W) @ Y.T
    Sg = S.cpu().numpy()
    assert np.max(np.abs(Sg - S_e)) <= 1e-12 * np.max(np.diag(S_e))
