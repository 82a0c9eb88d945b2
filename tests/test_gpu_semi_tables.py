"""Semianalytical estimator, wave per vertex: every depth of the bin search,
remainders of tiles, Philox blocks and samples, empty and tiny bins, and the
sample counts on both sides of the rule that keeps a thread per vertex."""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_18015_amd as cp
import workloads
from paper_2407_18015_amd import _lib as L

pytestmark = pytest.mark.gpu
HST = L.CP_HISTOGRAM


@pytest.mark.parametrize("H,W,nb,ns", [(9, 17, 2, 130), (16, 5, 4, 133), (7, 9, 5, 1001), (33, 20, 8, 129),
                                       (5, 70, 9, 258), (12, 12, 16, 255), (6, 6, 17, 400), (3, 3, 32, 511),
                                       (1, 9, 1, 128), (128, 257, 10, 140), (300, 300, 10, 66), (300, 300, 10, 67)])
@pytest.mark.parametrize("dtype,tol", [(torch.float32, 1e-6), (torch.float64, 1e-12)])
def test_semi_tables(H, W, nb, ns, dtype, tol):
    p = workloads.random_params(HST, 51, H, W, nbins=nb, width=0.15)
    rng = np.random.default_rng(52)
    kind = rng.random((nb, H, W))
    m = np.where(kind < 0.3, 0.0, np.where(kind < 0.4, 1e-9, p[2:]))
    m[rng.integers(0, nb, (H, W)), np.arange(H)[:, None], np.arange(W)[None]] += 0.1
    p[2:] = m / m.sum(0)
    pt = torch.as_tensor(np.ascontiguousarray(p), dtype=dtype, device="cuda")
    out = cp.semianalytical(pt, cp.field_of(pt, HST, nb, nsamples=ns, seed=(1 << 40) + 7, field_id=3), terms=True)
    idx = np.arange(H * W) if H * W < 800 else np.unique(np.r_[np.arange(0, H * W, 113), H * W - 5:H * W])
    ref = oracle.semi_at(pt.cpu().numpy().astype(np.float64), idx, ns, (1 << 40) + 7, 3)
    got = [out["min"], out["max"], out["terms"][0], out["terms"][1]]
    for k, g in enumerate(got):  # the estimator's parity bound
        d = np.abs(g.cpu().numpy().ravel()[idx] - ref[:, k])
        assert d.max() <= tol, (k, d.max())
