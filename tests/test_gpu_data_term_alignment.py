"""A data term that starts at any float (a view one element into a buffer): the solvers that read it
two pixels at a time give the same bits as from an aligned copy."""
import numpy as np
import pytest
import torch

from synth import make_small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,q", [(64, 3), (512, 2), (72, 2)])
def test_same_bits(n, q):
    import paper_1112_1805_amd as pkg
    w = make_small(n, q, 2, seed=n, lam=0.1, iters=3)
    plan = pkg.Plan(n, 1, q, 2)
    s = torch.empty((q, n, n), device="cuda:0")
    plan.datacost(torch.from_numpy(w.img.astype(np.float32)).to("cuda:0"), w.codebook, s)
    shifted = torch.empty(q * n * n + 1, device="cuda:0")[1:].view(q, n, n)
    shifted.copy_(s)
    assert shifted.data_ptr() % 8 == 4
    h = torch.empty((w.iters, 4), dtype=torch.float64, device="cuda:0")
    for run in (lambda x, u: plan.solve(x, plan.new_workspace(), w.lam, w.gamma, w.iters, u=u, hist=h),
                lambda x, u: plan.solve_pd(x, plan.new_workspace(), w.lam, 2.0, 0.5, w.iters, u=u, hist=h),
                lambda x, u: plan.solve_tv(x, plan.new_workspace(), 0.05, 1.0, w.iters, u=u, hist=h)):
        got = []
        for x in (s, shifted):
            u = torch.empty_like(s)
            run(x, u)
            got.append((u, h.clone()))
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
