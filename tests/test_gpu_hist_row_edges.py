"""Histogram adjoint with rows summed on chip, widths whose last 64-vertex tile holds
one to three vertices (a sweep wave of one lane, a gather vector across the tile's
edge): the first and the last rows against the oracle on the same rows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_18015_amd as cp
import workloads
from paper_2407_18015_amd import _lib as L

pytestmark = pytest.mark.gpu
HST = L.CP_HISTOGRAM


@pytest.mark.parametrize("H,W,nb,dtype", [(640, 577, 18, torch.float32), (640, 578, 18, torch.float32),
                                          (640, 579, 18, torch.float32), (560, 449, 13, torch.float64)])
def test_last_tile_of_few_vertices(H, W, nb, dtype):
    p = workloads.random_params(HST, 5, H, W, nbins=nb, width=0.06)
    rng = np.random.default_rng(5)
    t = [torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")
         for a in (p, rng.normal(size=(H, W)), rng.normal(size=(H, W)))]
    g = cp.backward(*t, cp.field_of(t[0], HST, nb)).cpu().numpy().astype(np.float64)
    rel, s = (1e-5, 5e-7) if dtype == torch.float32 else (1e-10, 1e-13)  # the parity bound of the adjoint
    for rows, keep in ((slice(0, 6), slice(0, 4)), (slice(H - 6, H), slice(2, 6))):
        a = [np.ascontiguousarray(u.cpu().numpy().astype(np.float64)[..., rows, :]) for u in t]
        ref, size = oracle.grad(HST, *a)[:, keep], oracle.grad(HST, *a, absolute=True)[:, keep]
        d = np.abs(g[:, rows][:, keep] - ref) - (rel * (1 + np.abs(ref)) + s * size)
        print(f"[parity] row edges {H}x{W}x{nb}: margin {d.max():.3e}", flush=True)
        assert d.max() <= 0
