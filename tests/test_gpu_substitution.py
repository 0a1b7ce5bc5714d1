"""Substitutions of orders 17..31 with a non-finite right-hand-side entry: the
unknowns solved before it is reached are the oracle's, in either direction."""
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
