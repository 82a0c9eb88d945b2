"""Histogram adjoint's gather at the widths around its vector: one vertex per
thread below it, whole vectors, a last vector that overlaps the one before; alone
and batched, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_18015_amd as cp
import workloads
from paper_2407_18015_amd import _lib as L

pytestmark = pytest.mark.gpu
HST = L.CP_HISTOGRAM


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_widths(dtype):
    rel, s = (1e-5, 5e-7) if dtype == torch.float32 else (1e-10, 1e-13)  # the parity bound of the adjoint
    fields, ps, ups, grads = [], [], [], []
    for H, W, nb in [(1, 1, 4), (3, 1, 4), (5, 2, 1), (4, 3, 10), (6, 4, 4), (1, 5, 4), (5, 6, 9), (4, 7, 4),
                     (9, 65, 4), (3, 129, 6), (1, 258, 4)]:
        p = workloads.random_params(HST, W, H, W, nbins=nb, width=0.06)
        rng = np.random.default_rng(W)
        up = [rng.normal(size=(H, W)) for _ in range(2)]
        dev = [torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda") for a in (p, *up)]
        fields.append(cp.field_of(dev[0], HST, nb))
        ps.append(dev[0])
        ups.append(dev[1:])
        grads.append(torch.empty_like(dev[0]))
        g = cp.backward(*dev, fields[-1])
        a = [t.cpu().numpy().astype(np.float64) for t in dev]
        ref, size = oracle.grad(HST, *a), oracle.grad(HST, *a, absolute=True)
        assert (np.abs(g.cpu().numpy() - ref) - (rel * (1 + np.abs(ref)) + s * size)).max() <= 0, (H, W, nb)
    cp.batched(fields, ps, gmin=[u[0] for u in ups], gmax=[u[1] for u in ups], grad=grads)
    for f, p, u, g in zip(fields, ps, ups, grads):
        assert torch.equal(g, cp.backward(p, *u, f)), (f.H, f.W)
