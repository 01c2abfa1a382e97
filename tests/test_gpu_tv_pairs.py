"""The TV solver's pixel kernels (two pixels per thread, compile-time label counts): every label
count, sides whose rows end inside a block, the storage types, a workspace full of NaN (the zero
start reads no state) and a stop by tolerance (w is written at checked iterations only), against
the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle.tvmodel as tvm
from synth import make_small

pytestmark = pytest.mark.gpu

# u against FP64 after a few iterations: FP32 arithmetic 2e-5; the 16-bit gradient state adds its
# rounding, 2^-11 (FP16) or 2^-8 (BF16) of values up to 1 + gamma lambda, averaged by the solve
TOL = {"f32": 2e-5, "f16": 2e-3, "bf16": 1.6e-2}


@pytest.mark.parametrize("n,q,store", [(64, q, "f32") for q in range(1, 9)] + [(72, 3, "f16"), (88, 8, "bf16"),
                                       (128, 5, "f16"), (360, 2, "f32"), (512, 7, "f16"), (64, 1, "bf16")])
def test_matches_oracle(n, q, store):
    import paper_1112_1805_amd as pkg
    iters, lam = 5, 0.05
    w = make_small(n, q, 2, seed=n + q, iters=iters)
    plan = pkg.Plan(n, 1, q, 2, store)
    print(n, q, store, flush=True)
    s = torch.empty((q, n, n), device="cuda:0")
    plan.datacost(torch.from_numpy(w.img.astype(np.float32)).to("cuda:0"), w.codebook, s)
    ref = tvm.tv_admm(s.cpu().numpy().astype(np.float64), float(np.float32(lam)), 1.0, iters)
    u = torch.empty_like(s)
    for hist in (None, torch.empty((iters, 4), dtype=torch.float64, device="cuda:0")):
        ws = plan.new_workspace()
        ws.fill_(0xff)
        st = plan.solve_tv(s, ws, lam, 1.0, iters, u=u, hist=hist)
        assert np.max(np.abs(u.cpu().numpy() - ref.w)) < TOL[store]
        assert np.isfinite(st["energy"])
    a = u.clone()
    ws.fill_(0xff)
    st = plan.solve_tv(s, ws, lam, 1.0, iters, u=u, tol=1e9, check_every=3)
    assert st["iters_done"] == 3
    ws.fill_(0xff)
    plan.solve_tv(s, ws, lam, 1.0, 3, u=a)
    assert torch.equal(a, u)
