"""Monte Carlo kernels at the edges of their work split: fields without some or
all neighbours (rows of the stencil matrix that repeat or drop out), sample
counts around the wave width, and vertex counts on both sides of the two-
vertices-per-wave rule (8192), odd ones among them, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_18015_amd as cp
import workloads
from paper_2407_18015_amd import _lib as L

pytestmark = pytest.mark.gpu

MVG = L.CP_MVGAUSS
CASES = [(1, 1, 100), (1, 2, 64), (1, 7, 63), (9, 1, 65), (2, 2, 1), (5, 6, 128), (64, 127, 40), (91, 91, 130)]


def setup(H, W):
    mem = workloads.correlated_ensemble(11, max(H, 8), max(W, 8))[:, :H, :W]
    return cp.fit(torch.as_tensor(np.ascontiguousarray(mem), dtype=torch.float32, device="cuda"), "mvg")


@pytest.mark.parametrize("H,W,ns", CASES)
def test_forward_edges(H, W, ns):
    params = setup(H, W)
    idx = np.arange(H * W) if H * W < 200 else np.unique(np.r_[np.arange(0, H * W, 97), H * W - 3:H * W])
    ref, amb = oracle.mvg_forward_at(params.cpu().numpy(), idx, ns, 77, 5)
    for est, cols in ((L.CP_MC_CONDITIONAL, (2, 3)), (L.CP_MC_HIT, (0, 1))):
        f = cp.Field(H, W, MVG, torch.float32, nsamples=ns, seed=77, field_id=5, estimator=est)
        for k, out in enumerate(cp.forward(params, f)):
            got, want = out.cpu().numpy().ravel()[idx].astype(np.float64), ref[:, cols[k]]
            if est == L.CP_MC_HIT:  # whole hits, equal but for the oracle's near-ties
                assert np.all(np.abs(np.rint(got * ns) - np.rint(want * ns)) <= amb[:, k]), k
            else:  # the parity bound of the estimator
                assert np.all(np.abs(got - want) <= 1e-6), (k, np.abs(got - want).max())


@pytest.mark.parametrize("H,W,ns", CASES)
def test_adjoint_edges(H, W, ns):
    params = setup(H, W)
    gmin, gmax = workloads.upstream(4, H, W)
    f = cp.Field(H, W, MVG, torch.float32, nsamples=ns, seed=78, field_id=6)
    g = cp.backward(params, *(torch.as_tensor(u, dtype=torch.float32, device="cuda") for u in (gmin, gmax)), f)
    idx = np.arange(H * W) if H * W < 200 else np.unique(np.r_[np.arange(0, H * W, 97), H * W - 3:H * W])
    ref, slack = oracle.mvg_grad_at(params.cpu().numpy(), gmin.astype(np.float64), gmax.astype(np.float64), idx, ns,
                                    78, 6, slack=True)
    got = g.cpu().numpy().reshape(16, -1).T[idx]
    # the parity bound of the adjoint: 2e-5 of the vertex's largest component, plus near-ties
    assert np.all(np.abs(got - ref) <= 2e-5 * (1 + np.abs(ref).max(1, keepdims=True)) + slack)


def test_adjoint_nan_neighbour():
    """A NaN mean reaches the gradient of the stencil whose first neighbour it is; a later neighbour's is skipped,
    as in the minimum."""
    params = setup(5, 6)
    params[0, 2, 3] = float("nan")
    one = torch.ones((5, 6), device="cuda")
    g = cp.backward(params, one, one, cp.Field(5, 6, MVG, torch.float32, nsamples=70, seed=1)).cpu().numpy()
    assert np.isnan(g[1, 2, 2]) and np.isnan(g[11:16, 2, 2]).all() and (g[2:11, 2, 2] == 0).all()
    assert np.isfinite(g[1:, 3, 3]).all()
