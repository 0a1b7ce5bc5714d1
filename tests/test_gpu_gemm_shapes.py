"""GEMM at wave scope over every transpose, at shapes around its 16-wide tiles
and 16-byte pieces, on operands on and off 16-byte alignment, against the
float64 product: the library's relative error bar, guard bands untouched, and
a non-finite row or column of an operand reaching only its own row or column
of C.  A^T A of one array (the route that loads it once) gives the bits of the
same product on two copies."""
import numpy as np
import pytest

from helpers import TOL, guarded, guards_intact, normwise

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (1, 3, 2), (3, 1, 5), (2, 16, 3), (7, 7, 13), (15, 16, 17), (16, 5, 4), (17, 33, 15), (30, 1, 64),
          (4, 1, 1), (5, 1, 64), (16, 1, 33), (17, 1, 9), (32, 1, 64), (33, 1, 40), (63, 1, 17), (64, 1, 64), (30, 30, 64), (31, 2, 49), (33, 48, 32), (48, 63, 1), (49, 18, 61), (64, 64, 64), (64, 13, 3), (63, 61, 62)]


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2609_28179_amd import glass
    return glass, torch


def _stored(a, t):
    return np.ascontiguousarray(np.swapaxes(a, 1, 2)) if t else a


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_wave_shapes(env, m, n, k, ta, tb):
    glass, torch = env
    print(f"gemm wave m={m} n={n} k={k} ta={ta} tb={tb}", flush=True)
    rng = np.random.default_rng([m, n, k, ta, tb])
    batch, alpha, beta = 21, -0.75, 1.25
    A, B, C = (rng.uniform(-1, 1, s).astype(np.float32) for s in ((batch, m, k), (batch, k, n), (batch, m, n)))
    A[3, m // 2, k // 2] = np.nan   # row m // 2 of problem 3
    B[5, k // 2, n // 2] = np.inf   # column n // 2 of problem 5
    prod = np.matmul(A.astype(np.float64), B.astype(np.float64))
    rows, cols = np.arange(m) != m // 2, np.arange(n) != n // 2
    for pad in (64, 65):
        (_, Ad), (_, Bd) = (guarded(torch, _stored(x, t), "cuda:0", pad) for x, t in ((A, ta), (B, tb)))
        for b in (0.0, beta):
            ref = alpha * prod + (b * C if b else 0.0)
            Cf, Cd = guarded(torch, C, "cuda:0", pad)
            assert glass.glass_gemm_batched_ex(ta, tb, m, n, k, batch, alpha, Ad, Bd, b, Cd, ("wave", 4)) == 0
            torch.cuda.synchronize()
            got = Cd.cpu().numpy()
            ok = [i for i in range(batch) if i not in (3, 5)]
            assert normwise(got[ok], ref[ok]).max() <= TOL
            assert np.isnan(got[3, m // 2]).all() and not np.isfinite(got[5, :, n // 2]).any()
            if rows.any():
                assert normwise(got[3:4, rows], ref[3:4, rows]).max() <= TOL
            if cols.any():
                assert normwise(got[5:6][:, :, cols], ref[5:6][:, :, cols]).max() <= TOL
            assert guards_intact(Cf, pad)


@pytest.mark.parametrize("n,k", [(1, 1), (7, 13), (16, 16), (30, 64), (33, 50), (64, 64), (63, 7)])
def test_one_array_as_both_operands(env, n, k):
    glass, torch = env
    print(f"gemm A^T A n={n} k={k}", flush=True)
    rng = np.random.default_rng([n, k])
    batch = 19
    J = torch.from_numpy(rng.uniform(-1, 1, (batch, k, n)).astype(np.float32)).to("cuda:0")
    J2, C1, C2 = J.clone(), torch.empty((batch, n, n), device="cuda:0"), torch.empty((batch, n, n), device="cuda:0")
    for b_, c in ((J, C1), (J2, C2)):
        assert glass.glass_gemm_batched_ex(1, 0, n, n, k, batch, 1.0, J, b_, 0.0, c, ("wave", 2)) == 0
    torch.cuda.synchronize()
    assert torch.equal(C1, C2)
    h = J.cpu().numpy().astype(np.float64)
    assert normwise(C1.cpu().numpy(), np.matmul(np.swapaxes(h, 1, 2), h)).max() <= TOL
