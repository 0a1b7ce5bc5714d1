"""POSV out of place: the bits of the in-place call at every scope, inputs left
as they were, B passed through where the factorization fails, and the
autograd forward on top of it."""
import numpy as np
import pytest

from paper_2609_28179_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2609_28179_amd import glass
    return glass, torch


@pytest.mark.parametrize("scope", ["thread", "wave", "workgroup", "subwave"])
@pytest.mark.parametrize("n,r", [(1, 1), (4, 3), (7, 1), (12, 9), (16, 1), (17, 1), (24, 5), (25, 1), (32, 2), (33, 1),
                                 (48, 17), (50, 1), (64, 1), (64, 33)])
def test_matches_in_place(env, scope, n, r):
    glass, torch = env
    if glass.glass_placement_feasible(glass.OP_POSV, n, r, glass.SCOPES[scope], 1) != 1:
        pytest.skip("infeasible placement")
    print(f"posv out of place n={n} nrhs={r} {scope}", flush=True)
    batch = 131
    c = inputs.make_case("posv", n, batch, cfg=7, nrhs=r)
    c["A"][5, n - 1, n - 1] = -100.0    # fails at its last pivot
    A, B = (torch.from_numpy(c[k]).to("cuda:0") for k in ("A", "B"))
    L, X, A0, B0 = A.clone(), B.clone(), A.clone(), B.clone()
    glass.posv_(L, X, force=(scope, 1))
    L2, X2 = torch.full_like(A, float("nan")), torch.full_like(B, float("nan"))
    info = torch.full((batch,), -7, dtype=torch.int32, device="cuda:0")
    assert glass.glass_posv_to_batched(n, r, batch, A, B, L2, X2, info, (scope, 1)) == 0
    torch.cuda.synchronize()
    h = info.cpu().numpy()
    assert h[5] == n and (np.delete(h, 5) == 0).all()
    ok = [i for i in range(batch) if i != 5]
    assert torch.equal(L2[ok], L[ok]) and torch.equal(X2[ok], X[ok])
    assert torch.equal(A, A0) and torch.equal(B, B0)
    assert torch.equal(X2[5], B[5])


def test_autograd_forward_keeps_inputs(env):
    """Contiguous, expanded and transposed operands give the in-place result."""
    glass, torch = env
    from paper_2609_28179_amd.autograd import cholesky_solve
    c = inputs.make_case("posv", 12, 40, cfg=8, nrhs=2)
    A, B = (torch.from_numpy(c[k]).to("cuda:0") for k in ("A", "B"))
    A0, B0 = A.clone(), B.clone()
    for a, b in ((A, B), (A[:1].expand(40, 12, 12), B), (A.transpose(1, 2), B.transpose(1, 2).contiguous().transpose(1, 2))):
        X = cholesky_solve(a, b)
        want = b.contiguous().clone()
        glass.posv_(a.contiguous().clone(), want)
        assert torch.equal(X, want)
    assert torch.equal(A, A0) and torch.equal(B, B0)
