"""Timed cases of the library: what its users call, through the public entry points.

A case is a dict of plain values.  "kind" names the calls of one pass, the
other entries their sizes and options:

  autograd      critical_point_probability and its gradient (a training step on a parameter field)
  fit_forward   fit_forward on an ensemble (fit and forward, fused where the layout allows)
  step          fit_forward, then the adjoint: the benchmark's step
  fit_then      fit, then forward as two calls
  classify      fit (or the error-bound fit), then all four class probabilities
  gauss         independent Gaussian: fit, classification, adjoint
  mvg           correlated Gaussian: fit, Monte Carlo forward
  mvg_adjoint   Monte Carlo adjoint on fitted parameters
  semi          semianalytical estimator on a fitted histogram field
  batched       many fields of uneven size, forward + adjoint, replayed graph

Fields are smooth sums of Gaussian bumps in [0, 1] with member noise, as the
benchmark's synthetic ensembles; everything is made on the GPU from the seed.
"""
import math

import torch

import paper_2407_18015_amd as cp

DTYPES = {"f32": torch.float32, "f64": torch.float64}
CONDITIONAL, HIT = 0, 1


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # a small parameter field in an optimisation loop (the repository's uniform FP64 64 x 64
        # configuration): launches and host work, not arithmetic
        {"name": "uniform_f64_64", "kind": "autograd", "model": "uniform", "dtype": "f64", "H": 64, "W": 64, "nbins": 0},
        # climate reanalysis after error-bounded compression (the paper's 240 x 960 sea-level pressure):
        # error-bound fit, then every vertex classified
        {"name": "climate_uniform_240x960", "kind": "classify", "model": "uniform", "dtype": "f32", "H": 240,
         "W": 960, "nbins": 0, "M": 1, "bound": True},
        # an ocean ensemble (the paper's Red Sea size, 20 members of 500 x 500), parametric model
        {"name": "ensemble_epa_500", "kind": "fit_forward", "model": "epanechnikov", "dtype": "f32", "H": 500,
         "W": 500, "nbins": 0, "M": 20},
        # the same ensemble with the nonparametric model at the paper's four bins
        {"name": "ensemble_hist4_500", "kind": "fit_then", "model": "histogram", "dtype": "f32", "H": 500, "W": 500,
         "nbins": 4, "M": 20},
        # the same ensemble with the correlated model at the paper's 2000 samples
        {"name": "ensemble_mvg_500x2000", "kind": "mvg", "model": "mvg", "dtype": "f32", "H": 500, "W": 500,
         "M": 20, "nsamples": 2000, "estimator": CONDITIONAL},
        # a double-precision study on an odd-sized crop (rows that no 16-byte load fits)
        {"name": "epa_f64_classify_723x1041", "kind": "classify", "model": "epanechnikov", "dtype": "f64", "H": 723,
         "W": 1041, "nbins": 0, "M": 12, "bound": False},
        # the benchmark's quoted step: fit + forward, then the adjoint, 20 members of 2048 x 2048
        {"name": "epa_step_2048", "kind": "step", "model": "epanechnikov", "dtype": "f32", "H": 2048, "W": 2048,
         "nbins": 0, "M": 20},
        # training through a large histogram field (the benchmark's 10 bins)
        {"name": "hist10_autograd_2048", "kind": "autograd", "model": "histogram", "dtype": "f32", "H": 2048,
         "W": 2048, "nbins": 10},
        # the independent Gaussian comparison model: fit, all classes, sensitivities
        {"name": "gauss_1024", "kind": "gauss", "model": "gaussian", "dtype": "f32", "H": 1024, "W": 1024, "M": 20},
        # sensitivities of the correlated model at the paper's 1000 samples
        {"name": "mvg_adjoint_512x1000", "kind": "mvg_adjoint", "model": "mvg", "dtype": "f32", "H": 512, "W": 512,
         "M": 20, "nsamples": 1000, "estimator": CONDITIONAL},
        # the sampled histogram estimator at the benchmark's 1000 samples
        {"name": "semi_hist10_1024x1000", "kind": "semi", "model": "histogram", "dtype": "f32", "H": 1024, "W": 1024,
         "nbins": 10, "M": 20, "nsamples": 1000},
        # a time series / multi-variable job: fields of uneven size and model in one call (the benchmark's
        # layout, sides 2^7..2^11, with fewer fields)
        {"name": "batched_18_fields", "kind": "batched", "model": "mixed", "dtype": "f32", "fields": 18, "layout": 0,
         "lo": 7.0, "hi": 11.0, "nbins": 10},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(2.0 ** rng.uniform(math.log2(lo), math.log2(hi))))))


def draw(rng):
    """One more case of the listed ranges: sizes log-uniform (odd ones among them), every model, type and bin count."""
    kind = rng.choice(["autograd", "classify", "fit_forward", "fit_then", "step", "gauss", "mvg", "mvg_adjoint",
                       "semi", "batched"])
    f64 = rng.random() < 0.3
    c = {"kind": kind, "dtype": "f64" if f64 else "f32"}
    if kind == "batched":
        c.update(model="mixed", fields=rng.randint(3, 18), layout=rng.randint(1, 10 ** 6), lo=6.0, hi=9.8 if f64 else 10.5,
                 nbins=rng.randint(3, 12))
        return c
    if kind in ("mvg", "mvg_adjoint"):
        c.update(model="mvg", dtype="f32", H=_log_int(rng, 40, 512), W=_log_int(rng, 40, 512), M=rng.randint(10, 40),
                 nsamples=_log_int(rng, 500, 2000),
                 estimator=HIT if kind == "mvg" and rng.random() < 0.25 else CONDITIONAL)
        return c
    if kind == "semi":
        c.update(model="histogram", H=_log_int(rng, 40, 1000), W=_log_int(rng, 40, 1000), nbins=rng.randint(3, 16),
                 M=rng.randint(10, 40), nsamples=_log_int(rng, 250, 1000))
        return c
    if kind == "gauss":
        top = 400 if f64 else 1024
        c.update(model="gaussian", H=_log_int(rng, 33, top), W=_log_int(rng, 33, top), M=rng.randint(10, 40))
        return c
    c["model"] = ("epanechnikov" if kind == "step" else rng.choice(["uniform", "epanechnikov"])
                  if kind == "fit_forward" else rng.choice(["uniform", "epanechnikov", "histogram"]))
    hist = c["model"] == "histogram"
    top = 1024 if hist or f64 else 2048
    c.update(H=_log_int(rng, 33, top), W=_log_int(rng, 33, top), nbins=rng.randint(3, 16) if hist else 0)
    if kind != "autograd":
        c["M"] = rng.randint(8, 40)
    if kind == "classify":
        c["bound"] = c["model"] == "uniform" and rng.random() < 0.5
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _base(g, H, W, dtype):
    """A sum of 64 separable Gaussian bumps, rescaled to [0, 1]."""
    dev = g.device
    u = torch.rand((4, 64), generator=g, device=dev, dtype=torch.float64)
    s = max(1.0, min(H, W) / 64.0) * (3.0 + 7.0 * u[3])
    gy = torch.exp(-(torch.arange(H, device=dev)[None] - H * u[1][:, None]) ** 2 / (2 * s[:, None] ** 2))
    gx = torch.exp(-(torch.arange(W, device=dev)[None] - W * u[2][:, None]) ** 2 / (2 * s[:, None] ** 2))
    f = ((2 * u[0] - 1)[:, None] * gy).T.contiguous() @ gx
    return ((f - f.min()) / (f.max() - f.min())).to(dtype)


def _members(g, kind, H, W, M, dtype):
    """[M, H, W]: smooth base plus member noise; "mixture" adds the two-component offset of the histogram
    workload, "correlated" smooths the noise over several cells."""
    base = _base(g, H, W, dtype)
    out = torch.empty((M, H, W), dtype=dtype, device=g.device)
    for k in range(M):
        n = torch.randn((H, W), generator=g, device=g.device, dtype=dtype)
        if kind == "smooth":
            n = torch.nn.functional.avg_pool2d(torch.nn.functional.pad(n[None], (2, 2, 2, 2), mode="replicate"), 5, 1)[0]
            out[k] = base + 0.05 * n
        elif kind == "correlated":
            for _ in range(3):
                n = torch.nn.functional.avg_pool2d(torch.nn.functional.pad(n[None], (3, 3, 3, 3), mode="replicate"), 7, 1)[0]
            out[k] = base + (0.05 / n.std()) * n
        else:
            c = (torch.rand((H, W), generator=g, device=g.device) < 0.3).to(dtype)
            out[k] = base + 0.3 * c + 0.05 * n
    return out


def _params(g, model, H, W, nbins, dtype):
    """A parameter field without an ensemble: smooth centre, per-vertex half-widths, random masses."""
    base = _base(g, H, W, torch.float64)
    wd = 0.005 + 0.015 * torch.rand((H, W), generator=g, device=g.device, dtype=torch.float64)
    if min(H, W) <= 128:
        wd = wd * 10.0  # steeper per cell: wider noise, as the small uniform configuration
    if model == "epanechnikov":
        return torch.stack([base, wd]).to(dtype)
    if model == "uniform":
        return torch.stack([base - wd, base + wd]).to(dtype)
    m = torch.rand((nbins, H, W), generator=g, device=g.device, dtype=torch.float64).clamp_min(1e-12).log().neg()
    return torch.cat([torch.stack([base - wd, base + wd]), m / m.sum(0)]).to(dtype)


def _layout(case):
    """(side, model) of a batched case's fields: part of the case, not of the seed."""
    g = torch.Generator().manual_seed(case["layout"])
    e = case["lo"] + (case["hi"] - case["lo"]) * torch.rand(case["fields"], generator=g, dtype=torch.float64)
    return [(int(round(2.0 ** float(v))), ("uniform", "epanechnikov", "histogram")[i % 3]) for i, v in enumerate(e)]


def _upstream(g, H, W, dtype):
    return [torch.randn((H, W), generator=g, device=g.device, dtype=dtype) for _ in range(2)]


def prepare(case, seed):
    g = torch.Generator(device=_device()).manual_seed(seed)
    kind, dt = case["kind"], DTYPES[case["dtype"]]
    s = {"case": case, "kind": kind, "seed": seed}
    if kind == "batched":
        s["fields"], s["params"], s["gmin"], s["gmax"] = [], [], [], []
        for side, model in _layout(case):
            p = _params(g, model, side, side, case["nbins"], dt)
            s["fields"].append(cp.field_of(p, model))
            s["params"].append(p)
            u = _upstream(g, side, side, dt)
            s["gmin"].append(u[0])
            s["gmax"].append(u[1])
        s["pmin"], s["pmax"] = ([torch.empty_like(u) for u in s["gmin"]] for _ in range(2))
        s["grad"] = [torch.empty_like(p) for p in s["params"]]
        return s
    H, W = case["H"], case["W"]
    if kind == "autograd":
        s["params"] = _params(g, case["model"], H, W, case["nbins"], dt).requires_grad_()
        s["up"] = _upstream(g, H, W, dt)
        return s
    noise = {"histogram": "mixture", "mvg": "correlated"}.get(case["model"], "smooth")
    s["members"] = _members(g, noise, H, W, case["M"], dt)
    if kind == "classify" and case["bound"]:
        s["field"] = s.pop("members")[0].contiguous()
        s["eb"] = 1e-3 * float(s["field"].max() - s["field"].min())
    if kind in ("step", "gauss", "mvg_adjoint"):
        s["up"] = _upstream(g, H, W, torch.float32 if case["model"] == "mvg" else dt)
    if kind == "mvg_adjoint":
        s["params"] = cp.fit(s.pop("members"), "mvg")
    if kind == "semi":
        s["params"] = cp.fit(s.pop("members"), "histogram", nbins=case["nbins"])
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    case, kind = s["case"], s["kind"]
    if kind == "batched":
        cp.batched(s["fields"], s["params"], pmin=s["pmin"], pmax=s["pmax"], gmin=s["gmin"], gmax=s["gmax"],
                   grad=s["grad"], graph=True)
        return {"pmin": s["pmin"], "pmax": s["pmax"], "grad": s["grad"]}
    model = case["model"]
    if kind == "autograd":
        pmin, pmax = cp.critical_point_probability(s["params"], model)
        (grad,) = torch.autograd.grad((pmin, pmax), s["params"], s["up"])
        return {"pmin": pmin, "pmax": pmax, "grad": grad}
    if kind == "fit_forward":
        params, pmin, pmax = cp.fit_forward(s["members"], model)
        return {"params": params, "pmin": pmin, "pmax": pmax}
    if kind == "step":
        params, pmin, pmax = cp.fit_forward(s["members"], model)
        grad = cp.backward(params, *s["up"], cp.field_of(params, model))
        return {"params": params, "pmin": pmin, "pmax": pmax, "grad": grad}
    if kind == "fit_then":
        params = cp.fit(s["members"], model, nbins=case["nbins"])
        pmin, pmax = cp.forward(params, cp.field_of(params, model))
        return {"params": params, "pmin": pmin, "pmax": pmax}
    if kind == "classify":
        if case["bound"]:
            params = cp.fit_error_bound(s["field"], s["eb"])
        else:
            params = cp.fit(s["members"], model, nbins=case["nbins"])
        return {"params": params, **cp.classify(params, cp.field_of(params, model))}
    if kind == "gauss":
        params = cp.fit(s["members"], model)
        f = cp.field_of(params, model)
        return {"params": params, **cp.classify(params, f), "grad": cp.backward(params, *s["up"], f)}
    if kind == "mvg":
        params = cp.fit(s["members"], model)
        f = cp.field_of(params, model, nsamples=case["nsamples"], seed=s["seed"], estimator=case["estimator"])
        pmin, pmax = cp.forward(params, f)
        return {"params": params, "pmin": pmin, "pmax": pmax}
    if kind == "mvg_adjoint":
        f = cp.field_of(s["params"], model, nsamples=case["nsamples"], seed=s["seed"])
        return {"grad": cp.backward(s["params"], *s["up"], f)}
    f = cp.field_of(s["params"], model, nsamples=case["nsamples"], seed=s["seed"])
    return cp.semianalytical(s["params"], f, terms=True)


# ---------------------------------------------------------------------------
# necessary work of one pass: inputs read once, outputs written once, and the
# arithmetic of an exact evaluation (a fused multiply-add counts 2)
# ---------------------------------------------------------------------------
# Per vertex, both sides, all pieces non-empty: per piece with k started
# neighbours n_k quadrature nodes (the smallest exact Gauss rules), 2 + 5k
# (uniform) or 6 + 7k (Epanechnikov) per node forward; about twice that with
# the leave-one-out products of the adjoint.
_FWD = {"uniform": 2 * (7 + 12 + 34 + 44 + 30), "epanechnikov": 2 * (39 + 80 + 162 + 238 + 60)}
_BWD = {"uniform": 2 * _FWD["uniform"], "epanechnikov": 2 * (57 + 136 + 294 + 448 + 90)}


def _closed(model, nbins):
    """(forward, adjoint, saddle) operations per vertex."""
    if model == "histogram":
        n = 5 * nbins  # merged sub-intervals of a stencil
        return 60 * n, 120 * n, 50 * n
    return _FWD[model], _BWD[model], _FWD[model]


def work(case):
    kind, el = case["kind"], 8 if case["dtype"] == "f64" else 4
    if kind == "batched":
        b = f = 0
        for side, model in _layout(case):
            n, q = side * side, 2 + (case["nbins"] if model == "histogram" else 0)
            b += n * el * (2 * q + 4)
            f += n * sum(_closed(model, case["nbins"])[:2])
        return {"bytes": b, "flops": f}
    n, model, M = case["H"] * case["W"], case["model"], case.get("M", 0)
    q = 2 + case.get("nbins", 0)
    if kind == "semi":
        # a quarter Philox block, the position, four tails and the four products of each sample
        return {"bytes": n * el * (q + 4), "flops": n * case["nsamples"] * 60}
    if kind == "mvg":
        # a Philox block, two Box-Muller pairs, the Cholesky product and two normal CDFs of each sample
        return {"bytes": n * (4 * M + 16 * 8 + 8), "flops": n * case["nsamples"] * 130}
    if kind == "mvg_adjoint":
        return {"bytes": n * (16 * 8 * 2 + 8), "flops": n * case["nsamples"] * 150}
    if kind == "gauss":
        # about 25 nodes resolve the product of five Gaussians in FP32 (50 in FP64), each four tails
        nodes = 50 if el == 8 else 25
        return {"bytes": n * el * (M + 2 + 4 + 2 + 2), "flops": n * (4 * M + nodes * 240)}
    fwd, bwd, sad = _closed(model, case["nbins"])
    if kind == "autograd":
        return {"bytes": n * el * (q + 2 + 2 + q), "flops": n * (fwd + bwd)}
    fit = 5 * M
    if kind == "step":
        return {"bytes": n * el * (M + q + 2 + 2 + q), "flops": n * (fit + fwd + bwd)}
    if kind == "classify":
        return {"bytes": n * el * (M + q + 4), "flops": n * (fit + fwd + sad)}
    return {"bytes": n * el * (M + q + 2), "flops": n * (fit + fwd)}


# ---------------------------------------------------------------------------
# the same values in 64 bits, in plain torch
# ---------------------------------------------------------------------------
_DY, _DX = (0, -1, 0, 1), (1, 0, -1, 0)  # e, n, w, s


def _gl(n, dev):
    """Gauss-Legendre nodes and weights by the eigenvalues of the Jacobi matrix."""
    k = torch.arange(1, n, dtype=torch.float64)
    b = k / torch.sqrt(4 * k * k - 1)
    x, v = torch.linalg.eigh(torch.diag(b, 1) + torch.diag(b, -1))
    return x.to(dev), (2 * v[0] ** 2).to(dev)


def _neighbours(p, r0, r1):
    """[4, ..., rows, W] neighbour values of rows r0..r1 of p [..., H, W] (absent: the vertex's own) and their
    presence [4, rows, W]."""
    H, W = p.shape[-2:]
    y = torch.arange(r0, r1, device=p.device)[:, None]
    x = torch.arange(W, device=p.device)[None]
    out, pres = [], []
    for dy, dx in zip(_DY, _DX):
        ok = (y + dy >= 0) & (y + dy < H) & (x + dx >= 0) & (x + dx < W)
        yy, xx = torch.where(ok, y + dy, y), torch.where(ok, x + dx, x)
        out.append(p[..., yy, xx])
        pres.append(ok)
    return torch.stack(out), torch.stack(pres)


def _products(S, F, pres):
    """prod S, prod F, S F S F, F S F S over the neighbours (first axis), absent ones 1, the mixed ones 0 where a
    neighbour is absent."""
    pr = pres.reshape(pres.shape + (1,) * (S.dim() - pres.dim()))
    one = torch.ones((), dtype=S.dtype, device=S.device)
    S, F = torch.where(pr, S, one), torch.where(pr, F, one)
    full = pr.all(0)
    return [S.prod(0), F.prod(0), S[0] * F[1] * S[2] * F[3] * full, F[0] * S[1] * F[2] * S[3] * full]


def _tails_ue(model, q, x):
    """S and F = 1 - S at x [rows, W, n] of distributions q [4, 2, rows, W]."""
    a, b = q[:, 0, ..., None], q[:, 1, ..., None]
    if model == "uniform":
        F = ((x - a) / (b - a)).clamp(0.0, 1.0)
        return 1.0 - F, F
    u = ((x - a) / b).clamp(-1.0, 1.0)
    return (1 - u) ** 2 * (2 + u) / 4, (1 + u) ** 2 * (2 - u) / 4


def _exact_ue(model, p, r0, r1):
    """(P_min, P_max, t1, t2) of rows r0..r1: Gauss-Legendre, exact for the degree, between the sorted support ends."""
    q, pres = _neighbours(p, r0, r1)
    v = p[:, r0:r1]
    lo = lambda z: z[..., 0, :, :] if model == "uniform" else z[..., 0, :, :] - z[..., 1, :, :]  # noqa: E731
    hi = lambda z: z[..., 1, :, :] if model == "uniform" else z[..., 0, :, :] + z[..., 1, :, :]  # noqa: E731
    a, b = lo(v), hi(v)
    e = torch.cat([lo(q), hi(q)]).permute(1, 2, 0)
    e = torch.minimum(torch.maximum(e, a[..., None]), b[..., None]).sort(-1).values
    e = torch.cat([a[..., None], e, b[..., None]], -1)
    gx, gw = _gl(8, p.device)
    hl, mid = (e[..., 1:] - e[..., :-1]) / 2, (e[..., 1:] + e[..., :-1]) / 2
    x = (mid[..., None] + hl[..., None] * gx).flatten(-2)
    w = (hl[..., None] * gw).flatten(-2)
    if model == "uniform":
        w = w / (b - a)[..., None]
    else:
        w = w * 0.75 / v[1][..., None] * (1 - ((x - v[0][..., None]) / v[1][..., None]) ** 2)
    return [(w * f).sum(-1) for f in _products(*_tails_ue(model, q, x), pres)]


def _exact_hist(p, r0, r1):
    """The same for histograms: every factor is linear between the merged bin edges (three nodes are exact)."""
    h = p.shape[0] - 2
    ends = p[:2].detach()
    q, pres = _neighbours(torch.cat([ends, p[2:]]), r0, r1)
    v = p[:, r0:r1]
    lo, hi = ends[0, r0:r1], ends[1, r0:r1]
    k = torch.arange(h + 1, device=p.device, dtype=p.dtype) / h
    edges = lambda l, u: l[..., None] + (u - l)[..., None] * k  # noqa: E731
    e = torch.cat([edges(lo, hi)] + [edges(q[i, 0].detach(), q[i, 1].detach()) for i in range(4)], -1)
    e = torch.minimum(torch.maximum(e, lo[..., None]), hi[..., None]).sort(-1).values
    gx, gw = _gl(3, p.device)
    hl, mid = (e[..., 1:] - e[..., :-1]) / 2, (e[..., 1:] + e[..., :-1]) / 2
    x = (mid[..., None] + hl[..., None] * gx).flatten(-2)
    w = (hl[..., None] * gw).flatten(-2)

    def at(l, u):
        z = (x - l[..., None]) * (h / (u - l))[..., None]
        j = z.floor().clamp(0, h - 1)
        return j.long(), (z - j).clamp(0.0, 1.0)

    jv, _ = at(lo, hi)
    w = w * v[2:].movedim(0, -1).gather(-1, jv) * (h / (hi - lo))[..., None]
    S, F = [], []
    for i in range(4):
        j, t = at(q[i, 0].detach(), q[i, 1].detach())
        m = q[i, 2:].movedim(0, -1)
        c = m.cumsum(-1)
        F.append((c - m).gather(-1, j) + m.gather(-1, j) * t)
        S.append(c[..., -1:] - F[-1])
    return [(w * f).sum(-1) for f in _products(torch.stack(S), torch.stack(F), pres)]


def _exact_gauss(p, up):
    """Composite Gauss-Legendre in vertex units, the gradient panel by panel."""
    H, W = p.shape[1:]
    dev = p.device
    gx, gw = _gl(10, dev)
    edges = torch.linspace(-9.0, 9.0, 61, dtype=torch.float64)
    out = [torch.zeros((H, W), dtype=torch.float64, device=dev) for _ in range(4)]
    leaf = p.clone().requires_grad_(up is not None)
    for a, b in zip(edges[:-1].tolist(), edges[1:].tolist()):
        q, pres = _neighbours(leaf, 0, H)
        t = (a + b) / 2 + (b - a) / 2 * gx
        x = leaf[0][..., None] + leaf[1][..., None] * t
        z = (x - q[:, 0, ..., None]) / q[:, 1, ..., None] * math.sqrt(0.5)
        f = _products(0.5 * torch.erfc(z), 0.5 * torch.erfc(-z), pres)
        w = (b - a) / 2 * gw * torch.exp(-t * t / 2) / math.sqrt(2 * math.pi)
        vals = [(w * v).sum(-1) for v in f]
        if up is not None:
            (vals[0] * up[0] + vals[1] * up[1]).sum().backward()
        for o, v in zip(out, vals):
            o += v.detach()
    return out, leaf.grad


def _exact_closed(model, p, up=None):
    """(P_min, P_max, t1, t2) of a parameter field in 64 bits and, with `up`, the gradient, some rows at a time."""
    p = p.detach().double()
    up = None if up is None else [u.double() for u in up]
    if model == "gaussian":
        return _exact_gauss(p, up)
    H, W = p.shape[1:]
    per = 40_000_000 // (W * (72 if model != "histogram" else 15 * (p.shape[0] - 1)))
    rows = max(1, per)
    leaf = p.clone().requires_grad_(up is not None)
    out = [torch.empty((H, W), dtype=torch.float64, device=p.device) for _ in range(4)]
    for r0 in range(0, H, rows):
        r1 = min(H, r0 + rows)
        v = _exact_hist(leaf, r0, r1) if model == "histogram" else _exact_ue(model, leaf, r0, r1)
        if up is not None:
            (v[0] * up[0][r0:r1] + v[1] * up[1][r0:r1]).sum().backward()
        for o, x in zip(out, v):
            o[r0:r1] = x.detach()
    return out, leaf.grad


def _exact_fit(case, s):
    """The fitted parameters in 64 bits; a later call is handed them in the field's type, so that is what its exact
    values are computed from (`.to`)."""
    model = case["model"]
    if case.get("bound"):
        d, h = s["field"].double(), 0.5 * s["eb"]
        return torch.stack([d - h, d + h])
    m = s["members"].double()
    if model == "uniform":
        return torch.stack([m.amin(0), m.amax(0)])
    if model in ("epanechnikov", "gaussian"):
        sd = m.std(0, correction=1)
        return torch.stack([m.mean(0), sd if model == "gaussian" else 1.06 * sd * case["M"] ** -0.2])
    if model == "histogram":
        # the bin of a member is decided in the field's type, every operation rounded once
        x, nb = s["members"], case["nbins"]
        lo, hi = x.amin(0), x.amax(0)
        j = ((x - lo) / (hi - lo) * nb).long().clamp(0, nb - 1)
        mass = torch.stack([(j == k).sum(0) for k in range(nb)]).double() / case["M"]
        return torch.cat([torch.stack([lo, hi]).double(), mass])
    # correlated Gaussian: mean, then the Cholesky factor of the stencil's covariance
    M, H, W = m.shape
    nb, pres = _neighbours(m, 0, H)
    x = torch.cat([nb, m[None]])
    x = x - x.mean(1, keepdim=True)
    pr = torch.cat([pres, torch.ones_like(pres[:1])]).movedim(0, -1)
    C = torch.stack([torch.stack([(x[a] * x[b]).sum(0) for b in range(5)], -1) for a in range(5)], -2) / (M - 1)
    eye = torch.eye(5, dtype=torch.float64, device=m.device)
    both = pr[..., :, None] & pr[..., None, :]
    L = torch.linalg.cholesky(torch.where(both, C + 1e-6 * eye, eye))
    return torch.stack([m.mean(0)] + [L[..., r, c] for r in range(5) for c in range(r + 1)])


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors holding 32-bit words."""
    lowmask = 0xFFFFFFFF
    k0, k1 = seed & lowmask, (seed >> 32) & lowmask
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (((p1 >> 32) & lowmask) ^ c1 ^ k0, p1 & lowmask, ((p0 >> 32) & lowmask) ^ c3 ^ k1,
                          p0 & lowmask)
        k0, k1 = (k0 + 0x9E3779B9) & lowmask, (k1 + 0xBB67AE85) & lowmask
    return c0, c1, c2, c3


def _u24(w):
    return ((w >> 8).double() + 0.5) * 2.0 ** -24


def _normals(w):
    r = torch.sqrt(-2.0 * torch.log(_u24(w[0])))
    a = 2.0 * math.pi * _u24(w[1])
    return r * torch.cos(a), r * torch.sin(a)


def _exact_mvg(case, p, seed, up=None):
    """The Monte Carlo estimate over the same samples, and its pathwise gradient."""
    H, W = p.shape[1:]
    n, ns, dev = H * W, case["nsamples"], p.device
    leaf = p.clone().requires_grad_(up is not None)
    nb, pres = _neighbours(p[:1], 0, H)
    ids = torch.arange(n, device=dev).reshape(H, W)
    near = torch.stack([_neighbours(ids[None], 0, H)[0][i, 0] for i in range(4)]).reshape(4, n)
    pres = pres.reshape(4, n, 1)
    acc = torch.zeros((2, n), dtype=torch.float64, device=dev)
    inf = torch.full((), math.inf, dtype=torch.float64, device=dev)
    per = max(1, (1 << (22 if up is not None else 24)) // n)
    for i0 in range(0, ns, per):
        i = torch.arange(i0, min(ns, i0 + per), device=dev)[None]
        flat = leaf.reshape(16, n)
        mu, L = flat[0], flat[1:, :, None]
        zero = torch.zeros_like(i)
        v = torch.arange(n, device=dev)[:, None]
        w = _philox(i + 0 * v, v + zero, zero, zero, seed)
        z = [*_normals(w[:2]), *_normals(w[2:])]
        tri = lambda r, k: sum(L[r * (r + 1) // 2 + c] * z[c] for c in range(k))  # noqa: E731
        x = torch.stack([(mu[near[r]] - mu)[:, None] + tri(r, r + 1) for r in range(4)])
        c = tri(4, 4)
        lo = torch.where(pres, x, inf).amin(0)
        hi = torch.where(pres, x, -inf).amax(0)
        if case["estimator"] == HIT:
            w = _philox(i + 0 * v, v + zero, zero, zero + 1, seed)
            xv = c + L[14] * _normals(w[:2])[0]
            e = [(xv < lo).double().sum(1), (xv > hi).double().sum(1)]
        else:
            e = [(0.5 * torch.erfc(-math.sqrt(0.5) * (lo - c) / L[14])).sum(1),
                 (0.5 * torch.erfc(-math.sqrt(0.5) * (c - hi) / L[14])).sum(1)]
        if up is not None:
            (sum((a * g.double().reshape(n)).sum() for a, g in zip(e, up)) / ns).backward()
        acc += torch.stack(e).detach()
    acc = (acc / ns).reshape(2, H, W)
    return (acc[0], acc[1]), leaf.grad


def _exact_semi(case, p, seed):
    p = p.double()
    H, W = p.shape[1:]
    n, ns, h, dev = H * W, case["nsamples"], case["nbins"], p.device
    q, pres = _neighbours(p, 0, H)
    q, pres, v = q.reshape(4, 2 + h, n), pres.reshape(4, n), p.reshape(2 + h, n)
    tab = lambda m: torch.cat([torch.zeros_like(m[:1]), m.cumsum(0)]).T.contiguous()  # noqa: E731
    cv, cn = tab(v[2:]), [tab(q[i, 2:]) for i in range(4)]
    T = cv[:, -1:]
    acc = [torch.zeros(n, dtype=torch.float64, device=dev) for _ in range(4)]
    ids = torch.arange(n, device=dev)[:, None]
    per = max(1, (1 << 23) // n)
    for b0 in range(0, (ns + 3) // 4, per):
        b = torch.arange(b0, min((ns + 3) // 4, b0 + per), device=dev)[None]
        w = torch.stack(_philox(b + 0 * ids, ids + 0 * b, torch.zeros_like(b), torch.zeros_like(b) + 2, seed), -1)
        keep = (4 * b[..., None] + torch.arange(4, device=dev) < ns).reshape(1, -1)
        r = _u24(w).reshape(n, -1) * T
        j = torch.zeros_like(r, dtype=torch.int64)
        for k in range(1, h):
            j += cv[:, k:k + 1] <= r
        c0 = cv.gather(1, j)
        m = cv.gather(1, j + 1) - c0
        f = torch.where(m > 0, ((r - c0) / m).clamp(0.0, 1.0), torch.zeros_like(r))
        x = (v[1] - v[0])[:, None] / h * (j + f)
        S, F = [], []
        for i in range(4):
            z = (x - (q[i, 0] - v[0])[:, None]) * (h / (q[i, 1] - q[i, 0]))[:, None]
            k = z.floor().clamp(0, h - 1)
            t = (z - k).clamp(0.0, 1.0)
            k = k.long()
            lo = cn[i].gather(1, k)
            F.append(lo + (cn[i].gather(1, k + 1) - lo) * t)
            S.append(cn[i][:, -1:] - F[-1])
        for a, e in zip(acc, _products(torch.stack(S), torch.stack(F), pres)):
            a += (e * keep).sum(1)
    return [(a * T[:, 0] / ns).reshape(H, W) for a in acc]


def exact(case, seed):
    s, kind = prepare(case, seed), case["kind"]
    model, dt = case["model"], DTYPES[case["dtype"]]
    if kind == "batched":
        each = [_exact_closed(m, p, (a, b))
                for (_, m), p, a, b in zip(_layout(case), s["params"], s["gmin"], s["gmax"])]
        return {"pmin": [v[0] for v, _ in each], "pmax": [v[1] for v, _ in each], "grad": [_mass(g) for _, g in each]}
    if kind == "autograd":
        v, g = _exact_closed(model, s["params"], s["up"])
        return {"pmin": v[0], "pmax": v[1], "grad": _mass(g)}
    if kind == "mvg_adjoint":
        return {"grad": _exact_mvg(case, s["params"], seed, s["up"])[1]}
    if kind == "semi":
        v = _exact_semi(case, s["params"], seed)
        return {"min": v[0], "max": v[1], "terms": torch.stack(v[2:])}
    fit = _exact_fit(case, s)
    if kind == "mvg":
        v, _ = _exact_mvg(case, fit, seed)
        return {"params": fit, "pmin": v[0], "pmax": v[1]}
    v, g = _exact_closed(model, fit.to(dt), s["up"] if kind in ("step", "gauss") else None)
    if kind in ("classify", "gauss"):
        sad = v[2] + v[3]
        out = {"params": fit, "min": v[0], "max": v[1], "saddle": sad, "regular": 1 - v[0] - v[1] - sad}
        return {**out, "grad": g} if kind == "gauss" else out
    out = {"params": fit, "pmin": v[0], "pmax": v[1]}
    return {**out, "grad": g} if kind == "step" else out


def _mass(g):
    """A parameter gradient in the library's layout: histogram ends are not differentiated (their planes are 0)."""
    if g.shape[0] > 2:
        g = g.clone()
        g[:2] = 0.0
    return g
