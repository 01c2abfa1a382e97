"""Performance cases of the segmentation library: what they call, on which inputs, and what a
correct result is.

Every case goes through the public binding (`paper_1112_1805_amd`): transforms, denoising, the
ADMM solver for one image and for a batch, and the primal-dual, TV and nonlocal solvers.  Sizes,
label counts, weights and image classes are those of `synth/workloads.py`, `bench.py` and the
tests; iteration counts are shorter than a full segmentation's (a solve is a repetition of one
iteration, and programs that show progress or checkpoint run it in pieces of this length).

Inputs are synthetic images of the classes the library is for: a curved Voronoi partition,
grey levels or random colours per label, oriented textures in half of the regions, Gaussian
noise.  Everything is made on the GPU from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1112_1805_amd as pkg

# --------------------------------------------------------------------------- the cases


def listed():
    return [
        # The smallest segmentation: thumbnails and previews.  Launches and latency count.
        {"name": "solve 128 gray f32", "kind": "solve", "n": 128, "channels": 1, "q": 3, "J": 2, "store": "f32",
         "iters": 64, "hist": True},
        # An ordinary grey image with textured regions, 16-bit state.
        {"name": "solve 512 gray f16", "kind": "solve", "n": 512, "channels": 1, "q": 4, "J": 3, "store": "f16",
         "iters": 40, "hist": False},
        # The headline workload: a 1024^2 colour image, five labels, 61 filters, with history.
        {"name": "solve 1024 rgb f16", "kind": "solve", "n": 1024, "channels": 3, "q": 5, "J": 4, "store": "f16",
         "iters": 24, "hist": True},
        # The largest image side and label count.
        {"name": "solve 2048 gray f16", "kind": "solve", "n": 2048, "channels": 1, "q": 8, "J": 4, "store": "f16",
         "iters": 10, "hist": True},
        # A cropped image whose side is no power of two, two labels (foreground / background).
        {"name": "solve 360 gray f16", "kind": "solve", "n": 360, "channels": 1, "q": 2, "J": 3, "store": "f16",
         "iters": 30, "hist": False},
        # A folder of images of different sizes and label counts, solved in one call.
        {"name": "batch 32 mixed f32", "kind": "batch", "count": 32, "lo": 96, "hi": 768, "step": 32, "qmax": 6,
         "J": 3, "store": "f32", "iters": 20, "pick": 3},
        # One transform of one small image: feature extraction, the shortest call.
        {"name": "forward 256 x1", "kind": "forward", "n": 256, "q": 1, "J": 3, "count": 1},
        # Reconstruction from edited coefficients, a ragged size, more images than the plan's group.
        {"name": "adjoint 736 x5", "kind": "adjoint", "n": 736, "q": 2, "J": 3, "count": 5},
        # Shrinkage denoising of a stack of images.
        {"name": "denoise 1024 x16", "kind": "denoise", "n": 1024, "q": 8, "J": 4, "count": 16},
        # The primal-dual alternative of the solver, full-precision dual variable.
        {"name": "pd 512 rgb f32", "kind": "pd", "n": 512, "channels": 3, "q": 6, "J": 3, "store": "f32",
         "iters": 30, "hist": True},
        # The comparison models of the paper: total variation and the nonlocal graph.
        {"name": "tv 1024 rgb f16", "kind": "tv", "n": 1024, "channels": 3, "q": 5, "J": 2, "store": "f16",
         "iters": 60, "hist": False},
        {"name": "nl 512 rgb f16", "kind": "nl", "n": 512, "channels": 3, "q": 5, "J": 2, "store": "f16",
         "iters": 60, "hist": False},
    ]


def _smooth(m):
    for p in (2, 3, 5, 7, 11, 13, 17, 19, 23):
        while m % p == 0:
            m //= p
    return m == 1


def _side(rng, lo, hi):
    """An image side the library takes: a power of two as often as any other multiple of 8,
    spread over the logarithm of [lo, hi]."""
    if rng.random() < 0.5:
        return 1 << rng.randint(math.ceil(math.log2(lo)), int(math.log2(hi)))
    while True:
        n = 8 * round(math.exp(rng.uniform(math.log(lo), math.log(min(hi, 1024)))) / 8)
        if lo <= n <= 1024 and _smooth(n):
            return n


def _scales(rng, n):
    return rng.randint(2, 4 if n >= 512 else 3)


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "batch", "forward", "adjoint", "denoise", "pd", "tv", "nl"])
    # the two state types in use: full precision, and FP16 for large images (BF16 is stored by
    # the same kernels with three bits less)
    store = rng.choice(["f32", "f16"])
    if kind == "batch":
        return {"kind": kind, "count": rng.randint(3, 32), "lo": 64, "hi": rng.choice([256, 512, 768]),
                "step": rng.choice([8, 32]), "qmax": 6, "J": 3, "store": store, "iters": rng.randint(4, 20),
                "pick": rng.randint(0, 999)}
    if kind in ("forward", "adjoint", "denoise"):
        n = _side(rng, 64, 1024)
        count = max(1, min(24, round(math.exp(rng.uniform(0.0, math.log(24.0 * max(1.0, (512 / n) ** 2)))))))
        return {"kind": kind, "n": n, "q": rng.randint(1, 8), "J": _scales(rng, n),
                "count": min(count, 4) if kind != "denoise" and n > 600 else count}
    if kind == "nl":
        n = _side(rng, 64, 512)
    elif kind == "solve":
        n = _side(rng, 64, 2048)
    else:
        n = _side(rng, 64, 1024)
    iters = rng.randint(6, 12) if n > 1024 else rng.randint(8, 30)
    q = rng.randint(2, 6 if n > 1024 else 8)
    return {"kind": kind, "n": n, "channels": rng.choice([1, 3]), "q": q,
            "J": rng.randint(2, 3) if kind in ("tv", "nl") else _scales(rng, n), "store": store, "iters": iters,
            "hist": rng.random() < 0.4}


def _shapes(case):
    """(n, q) of a batch's images, fixed by the case."""
    r = np.random.Generator(np.random.PCG64(31000 + case["pick"]))
    sides = [n for n in range(case["lo"], case["hi"] + 1, case["step"]) if _smooth(n)]
    return [(int(sides[r.integers(len(sides))]), int(r.integers(2, case["qmax"] + 1))) for _ in range(case["count"])]


# --------------------------------------------------------------------------- inputs

_DEV = "cuda:0" if torch.cuda.is_available() else "cpu"


def _gen(seed, stream=0):
    g = torch.Generator(device=_DEV)
    g.manual_seed(1_000_003 * int(seed) + stream)
    return g


def _image(n, channels, q, seed, stream=0):
    """A noisy image [channels][n][n] of q curved Voronoi regions and its codebook [q][channels]."""
    g = _gen(seed, stream)
    rnd = lambda *s: torch.rand(s, generator=g, device=_DEV)  # noqa: E731
    y, x = torch.meshgrid(torch.arange(n, device=_DEV, dtype=torch.float32),
                          torch.arange(n, device=_DEV, dtype=torch.float32), indexing="ij")
    ky, kx = (rnd(8) * 6 - 3) * (2 * math.pi / n), (rnd(8) * 6 - 3) * (2 * math.pi / n)
    ph = rnd(2, 8) * (2 * math.pi)
    dy, dx = torch.zeros_like(y), torch.zeros_like(x)
    for i in range(8):
        dy += 0.0075 * n * torch.sin(ky[i] * y + kx[i] * x + ph[0, i])
        dx += 0.0075 * n * torch.sin(kx[i] * y - ky[i] * x + ph[1, i])
    sites, best, lab = 24, torch.full_like(x, float("inf")), torch.zeros_like(x, dtype=torch.int64)
    pos = rnd(2, sites) * n
    for i in range(sites):
        d = (y + dy - pos[0, i]) ** 2 + (x + dx - pos[1, i]) ** 2
        lab = torch.where(d < best, torch.full_like(lab, i % q), lab)
        best = torch.minimum(d, best)
    if channels == 1:
        cb = torch.linspace(0.0, 1.0, q, device=_DEV)[:, None]
    else:
        cb = rnd(q, channels)
    img = cb[lab].permute(2, 0, 1).contiguous()
    period, theta, phase = 6 + 10 * rnd(q), math.pi * rnd(q), 2 * math.pi * rnd(q)
    wave = torch.sin(2 * math.pi * (x * torch.cos(theta)[lab] + y * torch.sin(theta)[lab]) / period[lab] + phase[lab])
    img = img + 0.1 * torch.where(lab % 2 == 1, wave, torch.zeros_like(wave))
    img = img + 0.1 * torch.randn(img.shape, generator=g, device=_DEV)
    return img.contiguous(), cb.cpu().numpy().astype(np.float32)


def _weights(J, channels=1):
    """Lambda and gamma: equal weights per scale for grey images of up to three scales (0.1 at
    two, 0.05 at three), the paper's texture weights at four, its noisy colour example's
    (gamma = 4) for colour images."""
    if channels > 1:
        return np.array([0.0, 0.1, 0.2, 0.4, 2.0][: J + 1], dtype=np.float32) / np.float32(100.0), 4.0
    if J <= 3:
        return np.array([0.0] + [0.1 if J == 2 else 0.05] * J, dtype=np.float32), 1.0
    return np.array([0.0, 0.1, 0.2, 0.4, 0.8], dtype=np.float32) / np.float32(20.0), 1.0


def _denoise_weights(J):
    return np.array([0.0, 0.03, 0.04, 0.06, 0.08][: J + 1], dtype=np.float32)


_TV_WEIGHT, _NL_WEIGHT, _PD_TAU, _PD_SIGMA = 0.05, 0.02, 2.0, 0.5


def _graph(img):
    """The nonlocal model's neighbour graph: an input of its solver, built once per image."""
    nbr, rev, degree = pkg.nl_graph(img.cpu().numpy())
    return torch.from_numpy(nbr).to(_DEV), torch.from_numpy(rev).to(_DEV), degree


def _stack(case, seed):
    return torch.cat([_image(case["n"], 1, 8, seed, 10 + i)[0] for i in range(case["count"])])


def _coefficients(case, seed):
    """Shearlet coefficients as an edit leaves them: sparse, mostly small, of every filter."""
    eta = pkg.shs_num_filters(case["J"])
    c = torch.randn((case["count"], eta, case["n"], case["n"]), generator=_gen(seed), device=_DEV)
    return c.mul_(c.abs()).mul_(0.1)


def _batch_data(case, seed):
    out = []
    for i, (n, q) in enumerate(_shapes(case)):
        img, cb = _image(n, 1, q, seed, 100 + i)
        out.append(((img - torch.from_numpy(cb).to(_DEV)[:, :, None]) ** 2).contiguous())
    return out


# --------------------------------------------------------------------------- the path


def prepare(case, seed):
    kind, f32 = case["kind"], dict(dtype=torch.float32, device=_DEV)
    if kind == "batch":
        shapes = [(n, 1, q, case["J"], case["store"]) for n, q in _shapes(case)]
        b = pkg.Batch(shapes)
        lam, gamma = _weights(case["J"])
        return {"case": case, "batch": b, "ws": b.new_workspace(), "s": _batch_data(case, seed),
                "lams": [lam] * len(shapes), "gammas": [gamma] * len(shapes),
                "u": [torch.empty((q, n, n), **f32) for n, q in _shapes(case)],
                "stats": torch.empty((len(shapes), 5), dtype=torch.float64, device=_DEV)}
    n, q, J = case["n"], case["q"], case["J"]
    if kind in ("forward", "adjoint", "denoise"):
        plan = pkg.Plan(n, 1, q, J)
        st = {"case": case, "plan": plan, "ws": plan.new_workspace()}
        if kind == "adjoint":
            st["c"] = _coefficients(case, seed)
            st["f"] = torch.empty((case["count"], n, n), **f32)
        else:
            st["f"] = _stack(case, seed)
            if kind == "forward":
                st["c"] = torch.empty((case["count"], plan.eta, n, n), **f32)
            else:
                st["out"] = torch.empty_like(st["f"])
        return st
    plan = pkg.Plan(n, case["channels"], q, J, case["store"])
    img, cb = _image(n, case["channels"], q, seed)
    st = {"case": case, "plan": plan, "ws": plan.new_workspace(), "img": img, "cb": cb,
          "s": torch.empty((q, n, n), **f32), "u": torch.empty((q, n, n), **f32),
          "hist": torch.empty((case["iters"], 4), dtype=torch.float64, device=_DEV) if case["hist"] else None}
    st["lam"], st["gamma"] = _weights(J, case["channels"])
    if kind == "nl":
        st["nbr"], st["rev"], st["degree"] = _graph(img)
    return st


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "batch":
        st["batch"].solve(st["s"], st["ws"], st["lams"], st["gammas"], case["iters"], u_list=st["u"], stats=st["stats"])
        return st["u"]
    plan, ws = st["plan"], st["ws"]
    if kind == "forward":
        return plan.shearlet_forward(st["f"], st["c"], ws)
    if kind == "adjoint":
        return plan.shearlet_adjoint(st["c"], st["f"], ws)
    if kind == "denoise":
        return plan.shearlet_denoise(st["f"], _denoise_weights(case["J"]), ws, out=st["out"])
    # a segmentation: data term, solve, statistics of the result
    s = plan.datacost(st["img"], st["cb"], st["s"])
    kw = dict(u=st["u"], hist=st["hist"])
    if kind == "solve":
        stats = plan.solve(s, ws, st["lam"], st["gamma"], case["iters"], **kw)
    elif kind == "pd":
        stats = plan.solve_pd(s, ws, st["lam"], _PD_TAU, _PD_SIGMA, case["iters"], **kw)
    elif kind == "tv":
        stats = plan.solve_tv(s, ws, _TV_WEIGHT, st["gamma"], case["iters"], **kw)
    else:
        step = 1.0 / math.sqrt(4.0 * st["degree"])
        stats = plan.solve_nl(s, st["nbr"], st["rev"], ws, _NL_WEIGHT, step, step, case["iters"], st["degree"], **kw)
    # The relaxed labelling (the label map is its argmax), the energy it was stopped at, and
    # the convergence history in the precision it is plotted in.
    return {"u": st["u"], "energy": stats["energy"],
            "hist": None if st["hist"] is None else st["hist"].float()}


# --------------------------------------------------------------------------- cost of a pass


def _solve_work(n, q, J, store, iters):
    eta, n2, sb = 1 + 4 * (2 ** J - 1), n * n, 4 if store == "f32" else 2
    # per iteration: the state read and written once; w, b_w read and written, s read
    return (iters * (2 * sb * eta * q * n2 + 20 * q * n2),
            iters * (2 * eta + 2) * q * 2.5 * n2 * math.log2(n2))


def work(case):
    kind = case["kind"]
    if kind == "batch":
        each = [_solve_work(n, q, case["J"], case["store"], case["iters"]) for n, q in _shapes(case)]
        return {"bytes": sum(e[0] for e in each), "flops": sum(e[1] for e in each)}
    n, q, J, n2 = case["n"], case["q"], case["J"], case["n"] ** 2
    eta, fft = 1 + 4 * (2 ** J - 1), 2.5 * n2 * math.log2(n2)
    if kind in ("forward", "adjoint"):
        return {"bytes": case["count"] * (1 + eta) * 4 * n2, "flops": case["count"] * (1 + eta) * fft}
    if kind == "denoise":
        return {"bytes": case["count"] * 8 * n2, "flops": case["count"] * (2 + 2 * eta) * fft}
    io = (case["channels"] + 2 * q) * 4 * n2
    sb, it = 4 if case["store"] == "f32" else 2, case["iters"]
    if kind in ("solve", "pd"):
        b, f = _solve_work(n, q, J, case["store"], it)
        return {"bytes": b + io, "flops": f + (1 + eta) * q * fft}
    if kind == "tv":
        # gradient state (2q images) and w, b_w read and written, s read; two real 2-D FFTs per label
        return {"bytes": it * q * n2 * (4 * sb + 20) + io, "flops": it * q * (2 * fft + 40 * n2)}
    # ten neighbours: dual variable read and written, graph (index and reverse) read, u read and written, s read
    return {"bytes": it * n2 * (20 * sb * q + 80 + 12 * q) + io, "flops": it * q * 10 * 10 * n2}


# --------------------------------------------------------------------------- 64-bit reference


def _v(x):
    x = x.clamp(0.0, 1.0)
    return x ** 4 * (35 - 84 * x + 70 * x ** 2 - 20 * x ** 3)


def _b(w):
    a = w.abs()
    out = torch.where((a >= 1) & (a <= 2), torch.sin(0.5 * math.pi * _v(a - 1)), torch.zeros_like(a))
    return torch.where((a > 2) & (a <= 4), torch.cos(0.5 * math.pi * _v(0.5 * a - 1)), out)


def _shear(a, b, j, k):
    a = torch.where(a == 0, torch.ones_like(a), a)
    r = a / 4.0 ** j
    w = 2.0 ** j * b / a + k
    return torch.sqrt(_b(2 * r) ** 2 + _b(r) ** 2) * torch.sqrt(_v(1 - w.abs()))


def _bank(n, J):
    """Every filter on the half grid [eta][n][n/2+1], float64 (Section 2 of the paper; order and
    Nyquist rule as include/shearseg.h documents them)."""
    idx = torch.arange(n, device=_DEV)
    om = torch.where(idx < (n + 1) // 2, idx, idx - n).double()
    o1, o2 = om[:, None].expand(n, n), om[None, :].expand(n, n)
    rho = 4.0 ** J / n
    x1, x2, a1, a2 = rho * o1, rho * o2, o1.abs(), o2.abs()
    zero = torch.zeros_like(x1)

    def filt(kind, j, k):
        if kind == 0:
            a = torch.maximum(x1.abs(), x2.abs())
            mid = torch.cos(0.5 * math.pi * _v(2 * a - 1))
            return torch.where(a <= 0.5, torch.ones_like(a), torch.where(a < 1, mid, zero))
        h = _shear(x1, x2, j, k)
        out = zero
        if kind != 2:
            out = out + torch.where(a2 < a1, h, zero)
        if kind != 1:
            out = out + torch.where(a1 < a2, _shear(x2, x1, j, k), zero)
        if kind == 3:
            out = out + torch.where((a1 == a2) & (a1 > 0), h, zero)
        return out

    kinds = [(0, 0, 0)]
    for j in range(J):
        ks = range(-(2 ** j - 1), 2 ** j)
        kinds += [(1, j, k) for k in ks] + [(2, j, k) for k in ks] + [(3, j, -(2 ** j)), (3, j, 2 ** j)]
    mirror = (-idx) % n
    edge = (idx[:, None] == n // 2) | (idx[None, :] == n // 2)
    bank = torch.empty((len(kinds), n, n // 2 + 1), dtype=torch.float64, device=_DEV)
    for i, kind in enumerate(kinds):
        p = filt(*kind)
        p = torch.where(edge, torch.sqrt(0.5 * (p ** 2 + p[mirror][:, mirror] ** 2)), p)
        bank[i] = p[:, : n // 2 + 1]
    return bank


_CHUNK = 8   # filters transformed at a time (memory)


def _forward(f, bank):
    F, n = torch.fft.rfft2(f), f.shape[-1]
    return torch.cat([torch.fft.irfft2(bank[j:j + _CHUNK] * F, s=(n, n)) for j in range(0, len(bank), _CHUNK)])


def _adjoint(c, bank):
    n, acc = c.shape[-1], 0.0
    for j in range(0, len(bank), _CHUNK):
        acc = acc + (bank[j:j + _CHUNK] * torch.fft.rfft2(c[j:j + _CHUNK])).sum(0)
    return torch.fft.irfft2(acc, s=(n, n))


def _simplex(g):
    """Projection of g [q][...] onto the probability simplex, by sorting."""
    q = g.shape[0]
    srt = torch.sort(g, dim=0, descending=True).values
    css = torch.cumsum(srt, dim=0) - 1
    k = torch.arange(1, q + 1, device=g.device, dtype=g.dtype).reshape([q] + [1] * (g.dim() - 1))
    rho = (srt - css / k > 0).sum(0, keepdim=True)
    return (g - torch.gather(css, 0, rho - 1) / rho).clamp_min(0.0)


def _per_filter(lam, J):
    return torch.tensor([float(lam[0])] + [float(lam[j + 1]) for j in range(J) for _ in range(4 << j)],
                        dtype=torch.float64, device=_DEV)[:, None, None]


def _energy(w, s, bank, lam):
    return float((w * s).sum()) + sum(float((lam * _forward(w[l], bank).abs()).sum()) for l in range(len(w)))


def _admm(s, bank, lam, gamma, iters):
    """Section 3's ADMM from the zero state: w^K and the history rows."""
    q = len(s)
    thr = gamma * lam
    clip = lambda x: torch.minimum(torch.maximum(x, -thr), thr)  # noqa: E731
    g = torch.zeros((q, len(bank)) + s.shape[1:], dtype=torch.float64, device=_DEV)   # b_v + S u
    w, bw, rows = torch.zeros_like(s), torch.zeros_like(s), []
    for _ in range(iters):
        u = torch.empty_like(s)
        dy = db = l1 = 0.0
        for l in range(q):
            b = clip(g[l])
            u[l] = 0.5 * (_adjoint(g[l] - 2 * b, bank) + (w[l] - bw[l]) - gamma * s[l])
            new = b + _forward(u[l], bank)
            nb = clip(new)
            dy += float((((new - nb) - (g[l] - b)) ** 2).sum())
            db += float(((nb - b) ** 2).sum())
            l1 += float((lam * (new - nb).abs()).sum())
            g[l] = new
        gw = bw + u
        wn = _simplex(gw)
        dy += float(((wn - w) ** 2).sum())
        db += float(((gw - wn - bw) ** 2).sum())
        w, bw = wn, gw - wn
        rows.append([math.sqrt(db), math.sqrt(dy) / gamma, dy + db, float((w * s).sum()) + l1])
    return w, rows


def _primal_dual(s, bank, lam, iters):
    q = len(s)
    y = torch.zeros((q, len(bank)) + s.shape[1:], dtype=torch.float64, device=_DEV)
    u, ubar, rows = torch.zeros_like(s), torch.zeros_like(s), []
    for _ in range(iters):
        g, dy, l1 = torch.empty_like(s), 0.0, 0.0
        for l in range(q):
            c = _forward(ubar[l], bank)
            new = torch.minimum(torch.maximum(y[l] + _PD_SIGMA * c, -lam), lam)
            dy += float(((new - y[l]) ** 2).sum())
            l1 += float((lam * c.abs()).sum())
            y[l] = new
            g[l] = u[l] - _PD_TAU * (_adjoint(new, bank) + s[l])
        un = _simplex(g)
        du = float(((un - u) ** 2).sum())
        rows.append([math.sqrt(du), math.sqrt(dy), du + dy, float((un * s).sum()) + l1])
        u, ubar = un, 2 * un - u
    return u, rows


def _grad(u):
    return torch.stack([torch.roll(u, -1, 1) - u, torch.roll(u, -1, 2) - u], 1)


def _ball(x, r):
    """Projection of every pixel's vector x [.., n, n] (all leading entries) onto the ball of radius r."""
    norm = torch.sqrt((x ** 2).flatten(0, -3).sum(0))
    return x * torch.where(norm > r, r / norm.clamp_min(1e-300), torch.ones_like(norm))


def _tv(s, weight, gamma, iters):
    q, n = s.shape[0], s.shape[-1]
    e = 4 * torch.sin(math.pi * torch.arange(n, device=_DEV, dtype=torch.float64) / n) ** 2
    inv = 1.0 / (1.0 + e[:, None] + e[None, : n // 2 + 1])
    r = gamma * weight
    g = torch.zeros((q, 2, n, n), dtype=torch.float64, device=_DEV)
    w, bw, rows = torch.zeros_like(s), torch.zeros_like(s), []
    for _ in range(iters):
        b = _ball(g, r)
        d = g - 2 * b
        rhs = (torch.roll(d[:, 0], 1, 1) - d[:, 0]) + (torch.roll(d[:, 1], 1, 2) - d[:, 1]) + (w - bw) - gamma * s
        u = torch.fft.irfft2(torch.fft.rfft2(rhs) * inv, s=(n, n))
        new = b + _grad(u)
        nb = _ball(new, r)
        gw = bw + u
        wn = _simplex(gw)
        dy = float((((new - nb) - (g - b)) ** 2).sum()) + float(((wn - w) ** 2).sum())
        db = float(((nb - b) ** 2).sum()) + float(((gw - wn - bw) ** 2).sum())
        l1 = weight * float(torch.sqrt(((new - nb) ** 2).flatten(0, 1).sum(0)).sum())
        g, w, bw = new, wn, gw - wn
        rows.append([math.sqrt(db), math.sqrt(dy) / gamma, dy + db, float((w * s).sum()) + l1])
    return w, rows, float((w * s).sum()) + weight * float(torch.sqrt((_grad(w) ** 2).flatten(0, 1).sum(0)).sum())


def _nonlocal(s, nbr, degree, weight, iters):
    q, n = s.shape[0], s.shape[-1]
    M, step = nbr.shape[0], 1.0 / math.sqrt(4.0 * degree)
    step = float(np.float32(step))
    j = nbr.reshape(M, -1).long()
    has = (j >= 0).double()[None]
    j0 = j.clamp_min(0)
    s2 = s.reshape(q, -1)
    D = lambda u: (u[:, j0.reshape(-1)].reshape(q, M, -1) - u[:, None]) * has  # noqa: E731
    Dt = lambda y: (torch.zeros_like(s2).index_add_(1, j0.reshape(-1), (y * has).reshape(q, -1))  # noqa: E731
                    - (y * has).sum(1))
    u, ubar, rows = torch.zeros_like(s2), torch.zeros_like(s2), []
    y = torch.zeros((q, M, n * n), dtype=torch.float64, device=_DEV)
    for _ in range(iters):
        z = D(ubar)
        new = y + step * z
        norm = torch.sqrt((new ** 2).sum((0, 1)))
        new = new * torch.where(norm > weight, weight / norm.clamp_min(1e-300), torch.ones_like(norm))
        un = _simplex(u - step * (Dt(new) + s2))
        dy, du = float(((new - y) ** 2).sum()), float(((un - u) ** 2).sum())
        rows.append([math.sqrt(du), math.sqrt(dy), du + dy,
                     float((un * s2).sum()) + weight * float(torch.sqrt((z ** 2).sum((0, 1))).sum())])
        y, u, ubar = new, un, 2 * un - u
    e = float((u * s2).sum()) + weight * float(torch.sqrt((D(u) ** 2).sum((0, 1))).sum())
    return u.reshape(s.shape), rows, e


def exact(case, seed):
    kind, J = case["kind"], case["J"]
    if kind == "batch":
        lam, gamma = _weights(J)
        return [_admm(s.double(), _bank(s.shape[-1], J), _per_filter(lam, J), gamma, case["iters"])[0]
                for s in _batch_data(case, seed)]
    n = case["n"]
    bank = None if kind in ("tv", "nl") else _bank(n, J)
    if kind == "forward":
        return torch.stack([_forward(f.double(), bank) for f in _stack(case, seed)])
    if kind == "adjoint":
        return torch.stack([_adjoint(c.double(), bank) for c in _coefficients(case, seed)])
    if kind == "denoise":
        lam, out = _per_filter(_denoise_weights(J), J), []
        for f in _stack(case, seed):
            c = _forward(f.double(), bank)
            out.append(_adjoint(c - torch.minimum(torch.maximum(c, -lam), lam), bank))
        return torch.stack(out)
    img, cb = _image(n, case["channels"], case["q"], seed)
    cb = torch.from_numpy(cb).to(_DEV).double()
    s = torch.stack([((img.double() - cb[k][:, None, None]) ** 2).sum(0) for k in range(case["q"])])
    lam, gamma = _weights(J, case["channels"])
    lam = _per_filter(lam, J)
    if kind == "solve":
        u, rows = _admm(s, bank, lam, gamma, case["iters"])
        energy = _energy(u, s, bank, lam)
    elif kind == "pd":
        u, rows = _primal_dual(s, bank, lam, case["iters"])
        energy = _energy(u, s, bank, lam)
    elif kind == "tv":
        u, rows, energy = _tv(s, float(np.float32(_TV_WEIGHT)), gamma, case["iters"])
    else:
        nbr, _, degree = _graph(img)
        u, rows, energy = _nonlocal(s, nbr, degree, float(np.float32(_NL_WEIGHT)), case["iters"])
    return {"u": u, "energy": energy,
            "hist": torch.tensor(rows, dtype=torch.float64) if case["hist"] else None}
