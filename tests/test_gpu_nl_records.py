"""The nonlocal solver's record layouts: every label count (16-bit records are padded to even
counts), both block bounds of the kernels and a graph whose dual variable does not fit the
state's place, against the FP64 oracle's iteration."""
import numpy as np
import pytest
import torch

import oracle.nlmodel as nlm
from oracle import datacost
from synth import make_small

pytestmark = pytest.mark.gpu

# state rounding of the dual variable: |y| <= lambda = 0.05 at relative 2^-11 / 2^-8, a few
# iterations with step 1/sqrt(4 degree) and up to 16 blocks
TOL = {"f32": 2e-6, "f16": 2e-4, "bf16": 2e-3}


@pytest.mark.parametrize("q", range(1, 9))
@pytest.mark.parametrize("m,J,store", [(5, 2, "f16"), (5, 2, "f32"), (8, 3, "bf16"), (8, 3, "f16"), (8, 3, "f32"),
                                       (2, 1, "f16")])
def test_matches_oracle(q, m, J, store):
    import paper_1112_1805_amd as pkg
    n, iters, lam = 64, 4, 0.05
    w = make_small(n, q, J, seed=q, iters=iters)
    img = w.img.astype(np.float32)
    nbr, rev, degree = pkg.nl_graph(img, m=m)
    step = 1.0 / np.sqrt(4.0 * degree)
    plan = pkg.Plan(n, 1, q, J, store)
    print(q, m, J, store, flush=True)
    s = torch.empty((q, n, n), device="cuda:0")
    plan.datacost(torch.from_numpy(img).to("cuda:0"), w.codebook, s)
    u = torch.empty_like(s)
    h = torch.empty((iters, 4), dtype=torch.float64, device="cuda:0")
    ws = plan.new_workspace()
    ws.fill_(0xff)                                       # the zero start reads no state
    plan.solve_nl(s, torch.from_numpy(nbr).to("cuda:0"), torch.from_numpy(rev).to("cuda:0"), ws, lam, step, step,
                  iters, degree, u=u, hist=h)
    ref = nlm.nl_primal_dual(s.cpu().numpy().astype(np.float64), nbr, lam, float(np.float32(step)),
                             float(np.float32(step)), iters)
    assert np.max(np.abs(u.cpu().numpy() - ref.u)) < TOL[store]
    assert np.all(np.isfinite(h.cpu().numpy()))
