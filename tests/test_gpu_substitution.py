"""The blocked kernels where they substitute (orders from 17 on): unknowns solved
before a non-finite right-hand-side entry is reached are the oracle's, and on
ill-conditioned systems factors and solutions are as accurate as those of a
plain FP32 substitution, which explicit inverses of diagonal blocks are not."""
import numpy as np
import pytest

import oracle
from helpers import TOL, normwise
from paper_2609_28179_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("trans", [0, 1])
def test_trsv_unknowns_before_a_nonfinite_entry(value, trans):
    import torch
    from paper_2609_28179_amd import glass
    fails = []
    for n in range(17, 32):
        at = sorted({1, 7, 15, 16, n - 2, n - 1} - {n})
        rng = inputs.rng_for(12, "trsv", n, len(at))
        L, x = inputs.lower_factor(rng, len(at), n), inputs.uniform(rng, (len(at), n))
        ref = oracle.trsv(L, x, trans)
        bad = x.copy()
        bad[np.arange(len(at)), at] = value
        for force in (None, ("wave", 1)):
            print(f"trsv n={n} trans={trans} entry {value} {force}", flush=True)
            Ld, xd = torch.from_numpy(L).to("cuda:0"), torch.from_numpy(bad).to("cuda:0")
            assert glass.glass_trsv_batched(n, len(at), trans, Ld, xd, force) == 0
            torch.cuda.synchronize()
            got = xd.cpu().numpy()
            for b, p in enumerate(at):
                s = slice(0, p) if trans == 0 else slice(p + 1, n)
                if got[b, s].size and not normwise(got[b:b + 1, s], ref[b:b + 1, s]).max() <= TOL:
                    fails.append((n, p, force))
                if np.isfinite(got[b, p]):
                    fails.append((n, p, force, "entry"))
    assert not fails, fails


# ------------------------------------------------ accuracy on condition 1e6
# Against FP32 references that substitute column by column.  Another order of
# the same operations leaves the error's size as it is, up to chance: the
# medians over 256 problems may differ by a quarter (each problem's error
# spreads by about two to one, a median of 256 of them by a tenth).
MARGIN = 1.25
KAPPA = 1e6
BATCH = 256


def _chol32(A):
    A, L = A.copy(), np.zeros_like(A)
    for j in range(A.shape[1]):
        L[:, j:, j] = A[:, j:, j] / np.sqrt(A[:, j, j])[:, None]
        A[:, j + 1:, j + 1:] -= L[:, j + 1:, j, None] * L[:, None, j + 1:, j]
    return L


def _rho_f(L, A):
    L = np.tril(L).astype(np.float64)
    return np.abs(np.matmul(L, np.swapaxes(L, 1, 2)) - A).max(axis=(1, 2)) / np.abs(A).max(axis=(1, 2))


@pytest.mark.parametrize("op", ["potrf", "posv"])
def test_factor_as_accurate_as_substitution(op):
    import torch
    from paper_2609_28179_amd import glass
    fails = []
    for n in range(17, 25):
        print(f"{op} n={n} condition {KAPPA:.0e}", flush=True)
        A = inputs.spd_conditioned(inputs.rng_for(13, "potrf", n, BATCH), BATCH, n, KAPPA)
        A64 = A.astype(np.float64)
        exact = np.linalg.cholesky(A64)
        Ad, Bd = torch.from_numpy(A).to("cuda:0"), torch.ones((BATCH, n, 1), device="cuda:0")
        info = torch.full((BATCH,), -7, dtype=torch.int32, device="cuda:0")
        if op == "potrf":
            assert glass.glass_potrf_batched(n, BATCH, Ad, info, ("wave", 1)) == 0
        else:
            assert glass.glass_posv_batched(n, 1, BATCH, Ad, Bd, info, ("wave", 1)) == 0
        torch.cuda.synchronize()
        got, ref = np.tril(Ad.cpu().numpy()), _chol32(A)
        assert (info.cpu().numpy() == 0).all()
        for name, f in (("error", lambda L: normwise(L, exact)), ("residual", lambda L: _rho_f(L, A64))):
            r = np.median(f(got)) / np.median(f(ref))
            if not r <= MARGIN:
                fails.append((n, name, round(float(r), 2)))
    assert not fails, fails
