"""Plans whose kernels pass 64 KB of LDS per block only with their static arrays counted: the
middle step at 2048^2 with seven labels (60,928 bytes dynamic, 8,832 static) and the column passes
at 616 and 624 (up to 64,896 and 1,280), against the FP64
oracle.  Tolerances as for the other solves: FP32 arithmetic over two iterations."""
import numpy as np
import pytest
import torch

import oracle
from synth import make_small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,q", [(616, 1), (624, 2), (2048, 7)])
def test_solve_matches_oracle(n, q):
    import paper_1112_1805_amd as pkg
    iters = 2
    w = make_small(n, q, 1, seed=n + q, lam=0.1, iters=iters)
    print(n, q, flush=True)
    plan = pkg.Plan(n, 1, q, 1)
    s = torch.empty((q, n, n), device="cuda:0")
    plan.datacost(torch.from_numpy(w.img.astype(np.float32)).to("cuda:0"), w.codebook, s)
    u = torch.empty_like(s)
    h = torch.empty((iters, 4), dtype=torch.float64, device="cuda:0")
    plan.solve(s, plan.new_workspace(), w.lam, w.gamma, iters, u=u, hist=h)
    so = oracle.datacost(w.img.astype(np.float32).astype(np.float64), w.codebook.astype(np.float32).astype(np.float64))
    r = oracle.admm(so, oracle.filter_bank(n, 1), oracle.lambda_per_filter(w.lam, 1), w.gamma, iters)
    assert np.max(np.abs(u.cpu().numpy() - r.w)) < 2e-5
    assert np.max(np.abs(h.cpu().numpy()[:, 2] - r.r_combined) / np.maximum(r.r_combined, 1e-30)) < 1e-4
