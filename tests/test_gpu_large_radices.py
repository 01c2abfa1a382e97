"""Every fused mixed-radix pass (ADMM, primal-dual and shrinkage rows, analysis, TV column solve)
at sides whose stage lists hold the largest radices, 17 to 24 in the row transform and up to 32 in
the column transform, on a first iteration (state not read) and later ones, against the FP64
oracle.  Tolerances as for the other mixed-radix sides: FP32 arithmetic over a few iterations."""
import numpy as np
import pytest
import torch

import oracle
from synth import make_small, random_image

pytestmark = pytest.mark.gpu


def f64(x):
    return np.asarray(x, np.float32).astype(np.float64)


@pytest.mark.parametrize("n", [136, 152, 184, 528, 552, 736, 768])
def test_solvers_match_oracle(n):
    import paper_1112_1805_amd as pkg
    q, J, iters, lam = 2, 2, 3, 0.05
    w = make_small(n, q, J, seed=n, lam=0.1, iters=iters)
    plan = pkg.Plan(n, 1, q, J)
    print(plan.describe(), flush=True)
    s = torch.empty((q, n, n), device="cuda:0")
    plan.datacost(torch.from_numpy(w.img.astype(np.float32)).to("cuda:0"), w.codebook, s)
    so, B, lam_f = oracle.datacost(f64(w.img), f64(w.codebook)), oracle.filter_bank(n, J), oracle.lambda_per_filter(w.lam, J)
    ws, u = plan.new_workspace(), torch.empty_like(s)
    h = torch.empty((iters, 4), dtype=torch.float64, device="cuda:0")

    r = oracle.admm(so, B, lam_f, w.gamma, iters)
    plan.solve(s, ws, w.lam, w.gamma, iters, u=u, hist=h)
    assert np.max(np.abs(u.cpu().numpy() - r.w)) < 2e-5
    assert np.max(np.abs(h.cpu().numpy()[:, 2] - r.r_combined) / r.r_combined) < 1e-4

    r = oracle.primal_dual(so, B, lam_f, 2.0, 0.5, iters)
    plan.solve_pd(s, ws, w.lam, 2.0, 0.5, iters, u=u, hist=h)
    assert np.max(np.abs(u.cpu().numpy() - r.u)) < 5e-5
    assert np.max(np.abs(h.cpu().numpy()[:, 1] - r.dy)) < 1e-4 * np.max(r.dy)

    r = oracle.tv_admm(so, lam, 1.0, iters)
    plan.solve_tv(s, ws, lam, 1.0, iters, u=u, hist=h)
    assert np.max(np.abs(u.cpu().numpy() - r.w)) < 5e-5
    assert np.max(np.abs(h.cpu().numpy()[:, 0] - r.r_primal)) < 1e-4 * np.max(r.r_primal)

    f = random_image(n, seed=n, channels=1).astype(np.float32)
    out = plan.shearlet_denoise(torch.from_numpy(f).to("cuda:0"), np.float32([0.0, 0.1, 0.2]), ws)
    ref = oracle.denoise(f64(f[0]), B, oracle.lambda_per_filter(f64([0.0, 0.1, 0.2]), J))
    assert np.linalg.norm(out[0].cpu().numpy() - ref) < 1e-5 * np.linalg.norm(f)
