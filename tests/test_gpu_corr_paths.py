"""GPU tests of the two launch forms of the correlation and the EWMA: one launch of 16 x 16 tiles for
small windows, 128 x 128 tiles in T slices above them. Sizes sit at tile edges, step remainders and on
both sides of the rule that chooses the form.

Tolerances, derived before the first run: with unit-variance rows a Gram entry over its norm is a sum of
T products of total absolute size at most 1 (Cauchy-Schwarz), so any summation order is within
(T + 8) 2^-53 of the exact value (8: means, norms, division), 1e-12 at T <= 4200; the EWMA's S has the
same bound relative to its largest variance."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1403_4099_amd import pga
from gpu_cases import say

pytestmark = pytest.mark.gpu

# the small form ends at N = 352 (T <= 4096) and N = 704 (T <= 1024)
SIZES = [(1, 2), (15, 3), (16, 16), (17, 127), (33, 129), (48, 1025), (352, 40), (353, 40), (704, 33), (705, 33),
         (353, 1025), (20, 4096), (20, 4097), (130, 4097)]


@pytest.mark.parametrize("N,T", SIZES, ids=[f"N{n}-T{t}" for n, t in SIZES])
def test_correlation_and_ewma_at_the_edges_of_both_forms(N, T):
    say(f"corr forms N={N} T={T}")
    rng = np.random.default_rng(N * 10007 + T)
    R = 0.5 * rng.standard_normal(T)[None, :] + rng.standard_normal((N, T))
    if N > 3:
        R[2] = 0.1                                    # constant, not a dyadic value: variance 0
    wide = torch.zeros((N, T + 3), dtype=torch.float64, device="cuda")     # rows not 16-byte aligned
    wide[:, :T] = torch.from_numpy(R)
    st = pga.new_status()
    C, hi, lo = pga.correlate(wide[:, :T], split=True, status=st)
    Cg = C.cpu().numpy()
    X = R - R.mean(axis=1, keepdims=True)
    if N > 3:
        X[2] = 0.0
    s = np.sqrt((X * X).sum(axis=1))
    with np.errstate(divide="ignore", invalid="ignore"):
        E = np.clip(np.where(np.outer(s, s) > 0, (X @ X.T) / np.outer(s, s), 0.0), -1.0, 1.0)
    np.fill_diagonal(E, 1.0)
    assert np.max(np.abs(Cg - E)) <= 1e-12
    assert np.array_equal(Cg, Cg.T) and np.all(np.diag(Cg) == 1.0)
    assert int(st[2]) == int((s == 0).sum())
    h_o, l_o = O.split_bf16(Cg)
    ld = pga.split_ld(N)
    for got, want in ((hi, h_o), (lo, l_o)):
        full = np.zeros((ld, ld), dtype=np.uint16)    # zero past N
        full[:N, :N] = want
        assert np.array_equal(got.cpu().numpy().view(np.uint16), full)

    S0 = X @ X.T / T + np.eye(N)
    for market in (False, True):
        S = torch.from_numpy(S0.copy()).cuda()
        C2, hi2, _ = pga.ewma(wide[:, :T], S, 0.97, market=market, split=True)
        Y = R - (R.mean(axis=0, keepdims=True) if market else 0.0)
        W = 0.03 * 0.97 ** np.arange(T - 1, -1, -1.0)
        S_e = 0.97 ** T * S0 + (Y * W) @ Y.T
        Sg, C2g = S.cpu().numpy(), C2.cpu().numpy()
        assert np.max(np.abs(Sg - S_e)) <= 1e-12 * np.max(np.diag(S_e))
        assert np.array_equal(Sg, Sg.T) and np.array_equal(C2g, C2g.T) and np.all(np.diag(C2g) == 1.0)
        d = np.sqrt(np.diag(Sg))
        assert np.max(np.abs(C2g - np.clip(Sg / np.outer(d, d), -1, 1))[~np.eye(N, dtype=bool)], initial=0.0) <= 1e-12
        assert np.array_equal(hi2.cpu().numpy().view(np.uint16)[:N, :N], O.split_bf16(C2g)[0])
