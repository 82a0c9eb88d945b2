"""Node rules of the independent-Gaussian quadrature against the oracle: the
trapezoidal rule where the sigmas of a stencil are comparable, the composite
Gauss-Legendre rule where a neighbour is much narrower, and the choice
between them.  The checkerboard gives every vertex neighbours of one ratio
rho = sigma_v / sigma_n (1 / rho on the other colour), so the sweep over rho
crosses the switch from either side; offsets of several sigmas put the
neighbours' supports partly or wholly outside the vertex's window, and an
offset of 0 makes all cuts of a stencil coincide."""
import numpy as np
import pytest
import torch
from scipy.special import erfc

import oracle
import paper_2407_18015_amd as cp
import workloads
from paper_2407_18015_amd import _lib as L

pytestmark = pytest.mark.gpu

_X, _W = np.polynomial.legendre.leggauss(20)
_DYX = ((0, 1), (-1, 0), (0, -1), (1, 0))  # e, n, w, s


def gradient(p, g1, g2):
    """The adjoint by 20-point panels of half a deviation of every
    distribution, in coordinates about the vertex and through the translation
    and scale invariances: the oracle integrates the vertex's own slots in
    data coordinates, and the rounding of those reaches 2e-7 at the narrowest
    sigma here."""
    _, H, W = p.shape
    grad = np.zeros_like(p)
    Phi = lambda z: 0.5 * erfc(-z / np.sqrt(2))
    pdf = lambda z: np.exp(-z * z / 2) / np.sqrt(2 * np.pi)
    for y in range(H):
        for x in range(W):
            nb = [(y + dy, x + dx) for dy, dx in _DYX if 0 <= y + dy < H and 0 <= x + dx < W]
            sv = p[1, y, x]
            d = np.array([p[0][v] - p[0, y, x] for v in nb])
            s = np.array([p[1][v] for v in nb])
            k = np.linspace(-9, 9, 37)
            e = np.unique(np.clip(np.concatenate([sv * k] + [a + b * k for a, b in zip(d, s)]), -9 * sv, 9 * sv))
            t = ((e[1:] + e[:-1])[:, None] / 2 + (e[1:] - e[:-1])[:, None] / 2 * _X).ravel()
            w = ((e[1:] - e[:-1])[:, None] / 2 * _W).ravel() * pdf(t / sv) / sv
            z = (t - d[:, None]) / s[:, None]
            for g, fac, sign in ((g1[y, x], Phi(-z), 1.0), (g2[y, x], Phi(z), -1.0)):
                own = np.zeros(2)
                for n, v in enumerate(nb):
                    f = w * pdf(z[n]) / s[n] * np.prod(np.delete(fac, n, 0), 0)
                    dm, ds = sign * f.sum(), sign * (f * z[n]).sum()
                    grad[(0, *v)] += g * dm
                    grad[(1, *v)] += g * ds
                    own -= dm, (d[n] * dm + s[n] * ds) / sv
                grad[:, y, x] += g * own
    return grad


RATIOS = (1.0, 2.0, 3.0, 4.0, 5.0, 6.0, 8.0, 12.0, 40.0, 3e3)


@pytest.mark.parametrize("offset", [0.0, 0.7, 4.0, 11.0])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_ratio_sweep(dtype, offset):
    """One 6 x 7 checkerboard per ratio, stacked; tolerances of the model's
    other tests: probabilities 1e-6 / 1e-12, gradients 1e-5 (1 + |g|) +
    5e-7 S / 1e-10 (1 + |g|) + 1e-13 S, S the sum of the magnitudes of the
    integrands of the terms added."""
    H, W = 6, 7
    yy, xx = np.mgrid[0:H, 0:W]
    odd = (yy + xx) % 2 == 1
    rng = np.random.default_rng(17)
    tol = 1e-6 if dtype == torch.float32 else 1e-12
    a, b = (1e-5, 5e-7) if dtype == torch.float32 else (1e-10, 1e-13)
    for rho in RATIOS:
        print(f"[case] gauss rules {dtype} offset {offset} rho {rho}", flush=True)
        sg = np.where(odd, 0.05 / rho, 0.05)
        mu = 0.3 + 0.05 * offset * odd * np.sign(rng.standard_normal((H, W)))
        p = torch.as_tensor(np.stack([mu, sg]), device="cuda").to(dtype)
        f = cp.field_of(p, L.CP_GAUSSIAN)
        out = cp.classify(p, f, terms=True)
        ph = p.cpu().numpy().astype(np.float64)
        ref = oracle.gauss(ph)
        for got, r in zip((out["min"], out["max"], out["terms"][0], out["terms"][1]), ref):
            assert np.abs(got.cpu().numpy() - r).max() <= tol, (rho, offset)
        g1, g2 = (g.astype(np.float32) for g in workloads.upstream(5, H, W))
        grad = cp.backward(p, *(torch.as_tensor(g, device="cuda").to(dtype) for g in (g1, g2)), f)
        u = [g.astype(np.float64) for g in (g1, g2)]
        gr = gradient(ph, *u)
        S = oracle.gauss_grad_at(ph, *u, np.arange(H * W), absolute=True).T.reshape(2, H, W)
        d = np.abs(grad.cpu().numpy() - gr)
        assert np.all(d <= a * (1 + np.abs(gr)) + b * S), (rho, offset, d.max())
