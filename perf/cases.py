"""The work whose speed is followed: what a user of this library has it do.

Every case is one pass through the public entry points of
``paper_2603_02059_amd.traknn`` on device-resident fields: neighbour search and
scores in each mode (whole matrix, bands, all lengths, fused, allocation-free),
the local intrinsic dimension, and the gradient of the scores. ``listed`` gives
the named cases, ``draw`` more of the same ranges, ``prepare`` a case's inputs
and the plan a program keeps, ``run`` one pass, ``work`` what a pass cannot do
without and ``exact`` its floating outputs in 64 bits by plain torch.

The fields are those of ``synth.py``, drawn on the GPU: smooth AR(1) noise with
an annual cycle, the 101300 Pa offset and planted dipoles; and, for the inputs
reduced to principal components, AR(1) series of decaying variance.
"""
import math

import torch

from paper_2603_02059_amd import traknn as tk

PRODUCTS = {"bf16x3": 3, "fp32": 1, "fp16": 1, "fp64": 1}
# Rough rates of the contraction (flop/s), only to bound what draw() asks for.
RATE = {"bf16x3": 1.3e15, "fp32": 1.4e14, "fp16": 1.0e15, "fp64": 2.0e13}


def listed():
    full = dict(T=27394, H=64, W=128, sigma=6.0, L=5, k=10)
    return [
        # the smallest call: a season and a half of a coarse grid, a kept plan
        dict(name="tiny_score", kind="score", T=512, H=32, W=32, sigma=3.0, L=3, k=5, prec="bf16x3"),
        # a serving loop that may not allocate: the fixed scratch's example size
        dict(name="serve_noalloc", kind="serve", T=2048, H=32, W=32, sigma=3.0, L=5, k=10, prec="bf16x3"),
        # a decade of an odd grid (ragged T and D) in plain FP32
        dict(name="decade_fp32", kind="score", T=3653, H=37, W=53, sigma=4.0, L=4, k=7, prec="fp32"),
        # training-like use: the autograd function, forward and backward
        dict(name="grad_small", kind="grad", T=1461, H=32, W=64, sigma=3.0, L=3, k=10, prec="bf16x3"),
        # attribution of the 100 rarest trajectories of 30 years: gradient alone,
        # from lists the program holds
        dict(name="backward_30y", kind="backward", T=10957, H=64, W=128, sigma=6.0, L=5, k=10, prec="bf16x3",
             weighted=100),
        # the headline: 75 years of daily fields
        dict(name="headline", kind="score", prec="bf16x3", **full),
        # the finer grid in one FP16 pass, the largest contraction
        dict(name="fine_grid_fp16", kind="score", T=27394, H=128, W=256, sigma=12.0, L=5, k=10, prec="fp16"),
        # all lengths 1..10 from one call
        dict(name="sweep_1_10", kind="sweep", prec="bf16x3", **{**full, "L": 10}),
        # the distance matrix streamed in bands
        dict(name="bands", kind="band", prec="bf16x3", rb=4088, **full),
        # a coarse grid with long lists, as for the intrinsic dimension study
        dict(name="small_grid_dim", kind="dim", T=27394, H=4, W=8, sigma=1.0, L=5, k=40, prec="bf16x3"),
        # the same grid, never storing the matrix
        dict(name="small_grid_fused", kind="fused", T=27394, H=4, W=8, sigma=1.0, L=5, k=10, prec="bf16x3"),
        # 13 principal components in the precision that needs no allowance
        dict(name="pca13_fused_fp64", kind="fused", T=27394, H=1, W=13, sigma=0.0, L=5, k=40, prec="fp64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(c):
    """Estimated seconds of a pass: the contraction and the passes over the matrix."""
    nl = c["L"] if c["kind"] == "sweep" else 1
    pairs = c["T"] * c["T"] / 2.0
    return PRODUCTS[c["prec"]] * 2.0 * c["H"] * c["W"] * pairs / RATE[c["prec"]] + 4e-12 * pairs * nl * (1 + c["k"] / 16.0)


def draw(rng):
    kind = rng.choice(["score", "score", "score", "serve", "grad", "backward", "sweep", "band", "dim", "fused", "fused"])
    prec = rng.choice(["bf16x3", "bf16x3", "bf16x3", "fp32", "fp16"])
    L = rng.randint(1, 12)
    k = _log_int(rng, 1, 50)
    T = _log_int(rng, 400, 27394)
    H, W = _log_int(rng, 4, 128), _log_int(rng, 8, 256)
    c = dict(kind=kind)
    if kind == "serve":
        T, H, W = _log_int(rng, 400, 2048), _log_int(rng, 4, 32), _log_int(rng, 8, 32)
    elif kind == "grad":
        T, H, W = _log_int(rng, 400, 10957), _log_int(rng, 8, 64), _log_int(rng, 8, 128)
    elif kind == "backward":
        T = _log_int(rng, 1461, 10957)
        c["weighted"] = _log_int(rng, 20, 400)
    elif kind == "sweep":
        L, k = rng.randint(2, 12), _log_int(rng, 1, 20)
    elif kind == "band":
        T = _log_int(rng, 2048, 27394)
        c["rb"] = 8 * max(1, int(T * rng.uniform(0.08, 0.5)) // 8)
    elif kind == "dim":
        H, W, k = _log_int(rng, 4, 8), _log_int(rng, 4, 8), rng.randint(20, 50)
        prec = "bf16x3" if prec == "fp16" else prec
    elif kind == "fused":
        if rng.random() < 0.5:
            prec, H, W = "fp64", 1, rng.randint(5, 40)
        else:
            H, W = _log_int(rng, 4, 32), _log_int(rng, 8, 64)
    sigma = 0.0 if H == 1 else max(1.0, 3.0 * H / 32.0)
    c.update(T=T, H=H, W=W, sigma=sigma, L=L, k=k, prec=prec)
    while _cost(c) > 0.02:  # the largest listed passes take 20 to 26 ms
        c["T"] = int(0.9 * c["T"])
    if kind == "serve":
        while tk.workspace_bytes(c["T"], H * W, L, L, k, prec) > tk.NOALLOC_MAX_BYTES:
            c["T"] = int(0.9 * c["T"])
    return c


def _circulant(n, sigma, device):
    """Periodic Gaussian smoothing of n cells (truncated at 4 sigma) as a
    matrix, each row of unit norm: smoothed unit noise has unit variance."""
    r = int(math.ceil(4.0 * sigma))
    taps = torch.zeros(n, dtype=torch.float64)
    for o in range(-r, r + 1):
        taps[o % n] += math.exp(-0.5 * (o / sigma) ** 2)
    taps /= taps.norm()
    return torch.stack([torch.roll(taps, i) for i in range(n)]).float().to(device)


def _ar1(e, phi=0.8):
    """AR(1) series of unit variance along dim 0 from unit noise, by doubling."""
    e[1:] *= math.sqrt(1.0 - phi * phi)
    s, f = 1, phi
    while f > 1e-9 and s < e.shape[0]:
        e[s:] += f * e[:-s].clone()
        s, f = 2 * s, f * f
    return e


def _fields(case, seed):
    """[T, H * W] float32 fields on the GPU, from the seed alone."""
    T, H, W, sigma, L = case["T"], case["H"], case["W"], case["sigma"], case["L"]
    dev = "cuda"
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    x = torch.randn((T, H * W), generator=g, device=dev)
    day = torch.arange(T, device=dev, dtype=torch.float64)
    season = torch.sin(2.0 * math.pi * day / 365.25).float()[:, None]
    if sigma <= 0.0:  # principal component scores
        std = 3e4 / torch.arange(1, W + 1, device=dev) ** 0.7
        x = _ar1(x) * std
        x[:, :1] += 2e4 * season
        return x.contiguous()
    if H > 1:
        A, B = _circulant(H, sigma, dev), _circulant(W, sigma, dev)
        x = (x.view(T * H, W) @ B).view(T, H, W).transpose(1, 2).reshape(T * W, H) @ A
        x = x.view(T, W, H).transpose(1, 2).reshape(T, H * W)
    x = _ar1(x.contiguous())
    x *= 1000.0
    x += 800.0 * season
    x += 101300.0
    n_ev = max(1, T // 1370)
    sd = W / 8.0
    pos = torch.rand((n_ev, 3), generator=g, device=dev).cpu().tolist()
    yy, xx = torch.meshgrid(torch.arange(H, device=dev), torch.arange(W, device=dev), indexing="ij")
    for i, (u, v, a) in enumerate(pos):  # one event in each n_ev-th of the series
        span = T // n_ev
        t0 = i * span + int(u * max(1, span - L))
        dy, dx = 1.5 * sd * math.sin(2 * math.pi * a), 1.5 * sd * math.cos(2 * math.pi * a)
        cy, cx = H / 2.0, W * (0.25 + 0.5 * v)
        lobe = lambda y, z: torch.exp(-0.5 * ((yy - y) ** 2 + (xx - z) ** 2) / sd ** 2)  # noqa: E731
        x[t0:t0 + L] += 4000.0 * (lobe(cy + dy, cx + dx) - lobe(cy - dy, cx - dx)).reshape(1, -1)
    return x


def _weights(case, seed):
    """Upstream weights of the scores, as a loss over all of them gives."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 1000003)
    n = case["T"] - case["L"] + 1
    return 0.5 + torch.rand(n, generator=g, device="cuda", dtype=torch.float64)


def _aligned(x):
    """The fields as the program keeps them: rows on 16 bytes (an odd grid's
    rows padded once, as the library asks of strided input)."""
    T, D = x.shape
    if D % 4 == 0:
        return x
    pad = torch.zeros((T, (D + 3) // 4 * 4), device=x.device)
    pad[:, :D] = x
    return pad[:, :D]


def _rarest(scores, n):
    w = torch.zeros_like(scores)
    w[torch.argsort(-scores)[:n]] = 1.0
    return w


def prepare(case, seed):
    kind, L, k, prec = case["kind"], case["L"], case["k"], case["prec"]
    X = _aligned(_fields(case, seed))
    T, D = X.shape
    st = {"case": case, "X": X}
    if kind == "grad":
        st["X"] = X.contiguous().requires_grad_(True)
        st["w"] = _weights(case, seed)
        return st
    if kind == "serve":
        st["plan"], _ = tk.traknn_plan(T, D, L, L, k, prec)
        n = T - L + 1
        st["idx"] = torch.empty((1, n, k), dtype=torch.int32, device="cuda")
        st["dist"] = torch.empty((1, n, k), dtype=torch.float64, device="cuda")
        st["scores"] = torch.empty((1, n), dtype=torch.float64, device="cuda")
        return st
    lmin = 1 if kind == "sweep" else L
    mode = "fused" if kind == "fused" else "matrix"
    st["plan"] = tk.Plan(T, D, lmin, L, k, prec, row_batch=case.get("rb", 0), mode=mode)
    if kind == "backward":
        idx, dist = st["plan"].knn(X)
        st["idx"], st["w"] = idx[0], _rarest(st["plan"].score(dist)[0], case["weighted"])
        st["plan"].release_workspace()
    return st


def run(state):
    case, X, p = state["case"], state["X"], state.get("plan")
    kind = case["kind"]
    if kind == "grad":
        s, idx = tk.score(X, case["L"], case["k"], case["prec"])
        grad, = torch.autograd.grad(s, X, grad_outputs=state["w"])
        return {"scores": s.detach(), "idx": idx, "grad": grad}
    if kind == "serve":
        tk.traknn_knn_noalloc(p, X, X.stride(0), state["idx"], state["dist"])
        tk.traknn_score(p, state["dist"], state["scores"])
        return {"idx": state["idx"], "dist": state["dist"], "scores": state["scores"]}
    if kind == "backward":
        return {"grad": p.backward(X, state["idx"], state["w"])}
    idx, dist = p.knn(X)
    out = {"idx": idx, "dist": dist}
    if kind == "dim":
        out["dim"] = p.local_dim(dist)
    else:
        out["scores"] = p.score(dist)
    return out


def work(case):
    T, D, L, k, kind = case["T"], case["H"] * case["W"], case["L"], case["k"], case["kind"]
    if kind == "backward":
        # the weighted windows, their neighbours' windows, and the gradient
        rows = min(T, case["weighted"] * (k + 1) * L)
        terms = 2.0 * case["weighted"] * k * L
        return {"bytes": 4.0 * D * (rows + T) + 12.0 * T + 4.0 * T * k, "flops": 3.0 * D * terms}
    nl = L if kind == "sweep" else 1
    rows = nl * T
    pairs = T * (T + 1) / 2.0
    b = 4.0 * T * D + rows * k * 12.0 + rows * (k if kind == "dim" else 1) * 8.0
    f = PRODUCTS[case["prec"]] * 2.0 * D * pairs + 2.0 * nl * pairs
    if kind == "grad":
        b += 4.0 * T * D + 8.0 * T
        f += 3.0 * D * 2.0 * T * k * L
    return {"bytes": b, "flops": f}


def _exact_lists(X, lmin, lmax, k):
    """Sorted k nearest (distances, indices) of every length, in 64 bits."""
    T = X.shape[0]
    Xc = X.double()
    Xc = Xc - Xc.mean(0)
    n2 = (Xc * Xc).sum(1)
    S = Xc @ Xc.t().contiguous()
    S.mul_(-2.0).add_(n2[:, None]).add_(n2[None, :]).clamp_(min=0.0)
    D = S.clone()
    np0 = T - lmin + 1
    dist = torch.full((lmax - lmin + 1, np0, k), math.inf, dtype=torch.float64, device=X.device)
    idx = torch.full((lmax - lmin + 1, np0, k), -1, dtype=torch.int64, device=X.device)
    for L in range(1, lmax + 1):
        n = T - L + 1
        if L > 1:  # D_L(i, j) = D_{L-1}(i, j) + d(i + L - 1, j + L - 1)
            D[:n, :n] += S[L - 1:, L - 1:]
        if L < lmin:
            continue
        for r0 in range(0, n, 4096):
            r1 = min(n, r0 + 4096)
            rows = D[r0:r1, :n].clone()
            off = torch.arange(n, device=X.device)[None, :] - torch.arange(r0, r1, device=X.device)[:, None]
            rows.masked_fill_(off.abs() < L, math.inf)
            v, j = torch.topk(rows, k, dim=1, largest=False, sorted=True)
            dist[L - lmin, r0:r1], idx[L - lmin, r0:r1] = v, j
    return dist, idx


def _exact_grad(X, idx, w, L, k):
    """Gradient of sum_t w_t s_t with the neighbour sets fixed, in 64 bits."""
    T = X.shape[0]
    A = torch.zeros((T, T), dtype=torch.float64, device=X.device)
    t = torch.nonzero(w).reshape(-1)
    tt = t[:, None].expand(-1, k).reshape(-1)
    jj = idx[t].reshape(-1)
    c = (w[t] / k)[:, None].expand(-1, k).reshape(-1)
    for m in range(L):
        A.index_put_((tt + m, jj + m), c, accumulate=True)
    A += A.t().clone()
    Xc = X.double()
    Xc = Xc - Xc.mean(0)
    return 2.0 * (A.sum(1)[:, None] * Xc - A @ Xc)


def exact(case, seed):
    kind, L, k = case["kind"], case["L"], case["k"]
    X = _fields(case, seed)
    lmin = 1 if kind == "sweep" else L
    dist, idx = _exact_lists(X, lmin, L, k)
    scores = dist.mean(2)
    scores[torch.isinf(scores)] = math.nan  # lengths with fewer trajectories
    if kind == "backward":
        w = _rarest(scores[0], case["weighted"])
        return {"grad": _exact_grad(X, idx[0], w, L, k)}
    if kind == "grad":
        return {"scores": scores[0], "idx": None, "grad": _exact_grad(X, idx[0], _weights(case, seed), L, k)}
    out = {"idx": None, "dist": dist}
    if kind == "dim":
        # the estimate of two nearly equal distances magnifies their rounding
        # without bound: no value to hold it to
        out["dim"] = None
    else:
        out["scores"] = scores
    return out
