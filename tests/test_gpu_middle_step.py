"""The middle step of a solver iteration (adjoint rows, pixel step, row transform in one kernel)
at the smallest and largest sides, every label count's corner (one label; all eight; counts that
do not divide a wave's rows) and sides that are no power of two, against the FP64 oracle; and the
first iteration's state, which is written without being read."""
import numpy as np
import pytest
import torch

import oracle
from synth import make_small

pytestmark = pytest.mark.gpu


def run(w, store="f32", pd=False, poison=False):
    import paper_1112_1805_amd as pkg
    plan = pkg.Plan(w.n, w.channels, w.q, w.J, store)
    s = torch.empty((w.q, w.n, w.n), device="cuda:0")
    plan.datacost(torch.from_numpy(w.img.astype(np.float32)).to("cuda:0"), w.codebook, s)
    ws = plan.new_workspace()
    if poison:
        ws.fill_(0xff)                       # NaN in every type
    u = torch.empty_like(s)
    h = torch.empty((w.iters, 4), dtype=torch.float64, device="cuda:0")
    if pd:
        plan.solve_pd(s, ws, w.lam, 2.0, 0.5, w.iters, u=u, hist=h)
    else:
        plan.solve(s, ws, w.lam, w.gamma, w.iters, u=u, hist=h)
    return u.cpu().numpy(), h.cpu().numpy()


@pytest.mark.parametrize("n,q,J,iters", [(64, 1, 2, 4), (64, 8, 2, 4), (128, 3, 2, 4), (256, 5, 2, 4), (512, 7, 2, 3),
                                         (1024, 8, 1, 2), (2048, 8, 1, 2), (72, 1, 2, 4), (72, 7, 2, 4), (88, 5, 2, 4),
                                         (360, 2, 2, 4), (440, 3, 2, 3), (1000, 8, 1, 2)])
def test_solve_matches_oracle(n, q, J, iters):
    w = make_small(n, q, J, seed=7 * n + q, lam=0.1, iters=iters)
    print(n, q, flush=True)
    s = oracle.datacost(w.img.astype(np.float32).astype(np.float64), w.codebook.astype(np.float32).astype(np.float64))
    r = oracle.admm(s, oracle.filter_bank(n, J), oracle.lambda_per_filter(w.lam, J), w.gamma, iters)
    u, h = run(w)
    # FP32 against FP64 over a few iterations of values up to about 1: 2e-5 as elsewhere
    assert np.max(np.abs(u - r.w)) < 2e-5
    assert np.max(np.abs(h[:, 2] - r.r_combined) / r.r_combined) < 1e-4


@pytest.mark.parametrize("n,store", [(64, "f16"), (512, "f32"), (72, "bf16"), (360, "f32")])
@pytest.mark.parametrize("pd", [False, True])
def test_first_iteration_reads_no_state(n, store, pd):
    w = make_small(n, 3, 2, seed=n, lam=0.1, iters=3)
    a, b = run(w, store, pd), run(w, store, pd, poison=True)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
