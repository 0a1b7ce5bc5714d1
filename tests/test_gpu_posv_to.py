"""POSV out of place: the bits of the in-place call at every scope, inputs left
as they were, B passed through where the factorization fails, and the
autograd forward on top of it."""
import numpy as np
import pytest

import oracle
from helpers import TOL, normwise
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


@pytest.mark.parametrize("r", [2, 3, 4, 5])
def test_several_columns_every_blocked_order(env, r):
    """POTRS with few right-hand sides at every order of the blocked kernels
    (up to four columns take the 4 x 4 x 1 products): against the oracle."""
    glass, torch = env
    fails = []
    for n in range(17, 65):
        c = inputs.make_case("potrs", n, 9, cfg=11, nrhs=r)
        L, B = (torch.from_numpy(c[k]).to("cuda:0") for k in ("L", "B"))
        assert glass.glass_potrs_batched(n, r, 9, L, B, ("wave", 1)) == 0
        torch.cuda.synchronize()
        err = normwise(B.cpu().numpy(), oracle.potrs(c["L"], c["B"])).max()
        if not err <= TOL:
            fails.append((n, err))
    assert not fails, fails


@pytest.mark.parametrize("n,r,batch", [(17, 2, 40000), (20, 4, 65536), (24, 5, 65536), (24, 1, 65536), (16, 2, 40000)])
def test_default_placement_several_columns(env, n, r, batch):
    """force = NULL on either side of the rule for several columns: the
    oracle's tolerance on a sample spread over the batch, info 0 throughout."""
    glass, torch = env
    c = inputs.make_case("posv", n, 512, cfg=12, nrhs=r)
    reps = -(-batch // 512)
    A, B = (torch.from_numpy(c[k]).to("cuda:0").repeat(reps, 1, 1)[:batch].contiguous() for k in ("A", "B"))
    info = torch.full((batch,), -7, dtype=torch.int32, device="cuda:0")
    assert glass.glass_posv_batched(n, r, batch, A, B, info) == 0
    torch.cuda.synchronize()
    pick = np.unique(np.r_[0:16, batch // 2:batch // 2 + 16, batch - 16:batch])
    _, X_ref, _ = oracle.posv(c["A"][pick % 512], c["B"][pick % 512])
    assert normwise(B.cpu().numpy()[pick], X_ref).max() <= TOL
    assert (info.cpu().numpy() == 0).all()


def test_autograd_forward_takes_negated_views(env):
    """A negated view shares the storage of the values it negates: the solve
    uses the values, for A, for B and in the gradients."""
    glass, torch = env
    from paper_2609_28179_amd.autograd import cholesky_solve
    c = inputs.make_case("posv", 6, 10, cfg=9, nrhs=2)
    A, B = (torch.from_numpy(c[k]).to("cuda:0") for k in ("A", "B"))
    want = cholesky_solve(A, B)
    nA, nB = torch._neg_view(-A), torch._neg_view(-B)
    assert nA.is_neg() and nB.is_neg() and nA.is_contiguous()
    assert torch.equal(cholesky_solve(nA, nB), want)
    a, b = A.clone().requires_grad_(), B.clone().requires_grad_()
    g = torch.autograd.grad(cholesky_solve(a, b).sum(), (a, b))
    n = torch.autograd.grad(cholesky_solve(torch._neg_view(-a), torch._neg_view(-b)).sum(), (a, b))
    assert torch.equal(g[0], n[0]) and torch.equal(g[1], n[1])
