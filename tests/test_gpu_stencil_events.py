"""Uniform and Epanechnikov stencils whose supports start and end in every
order: the pieces beside the centre and the centre itself of P_min, P_max, the
saddle terms and the adjoint, against the oracle.

"mixed": widths over a factor of fifty, FP64; "ties": centres and widths on a
grid of 1/8, so events coincide and centres are empty or a point; "apart":
supports a million widths apart beside overlapping ones."""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_18015_amd as cp

pytestmark = pytest.mark.gpu

H, W = 37, 70


def params(model, kind):
    rng = np.random.default_rng(5)
    m, w = rng.normal(0, 0.3, (H, W)), np.exp(rng.uniform(np.log(0.02), 0, (H, W)))
    if kind == "ties":
        m, w = rng.integers(-4, 5, (H, W)) / 8, rng.integers(1, 5, (H, W)) / 8
    if kind == "apart":
        w = np.full((H, W), 0.25)
        m = m + 2.0 ** 18 * rng.integers(0, 3, (H, W))
    p = np.stack([m - w, m + w] if model == 0 else [m, w])
    return p.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("model", [0, 1])
@pytest.mark.parametrize("kind,dtype,tol", [("mixed", torch.float64, 1e-12), ("ties", torch.float64, 1e-12),
                                            ("ties", torch.float32, 1e-6), ("apart", torch.float64, 1e-9)])
def test_stencil_events(model, kind, dtype, tol):
    p = params(model, kind)
    pt = torch.as_tensor(p, dtype=dtype, device="cuda")
    out = cp.classify(pt, cp.field_of(pt, model), terms=True)
    ref = [*oracle.forward(model, p), *(t.reshape(H, W) for t in oracle.saddle_at(model, p, np.arange(H * W)))]
    for k, (g, r) in enumerate(zip([out["min"], out["max"], *out["terms"]], ref)):
        d = np.abs(g.cpu().numpy() - r)
        assert d.max() <= tol, (k, d.max())  # the parity bounds; "apart" adds the rounding of 2^19 / 0.25 units


@pytest.mark.parametrize("model", [0, 1])
@pytest.mark.parametrize("kind", ["mixed", "ties"])
def test_stencil_events_adjoint(model, kind):
    p = params(model, kind)
    rng = np.random.default_rng(6)
    up = [rng.normal(size=(H, W)) for _ in range(2)]
    pt = torch.as_tensor(p, dtype=torch.float64, device="cuda")
    g = cp.backward(pt, *(torch.as_tensor(u, device="cuda") for u in up), cp.field_of(pt, model)).cpu().numpy()
    ref = oracle.grad(model, p, *up)
    size = oracle.grad(model, p, *up, absolute=True)
    # FP64 parity bound of the adjoint: 1e-12 of the summed magnitudes
    assert np.all(np.abs(g - ref) <= 1e-12 * (1 + np.abs(ref)) + 1e-12 * size)
