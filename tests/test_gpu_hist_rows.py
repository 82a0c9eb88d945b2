"""Histogram adjoint with rows summed on chip (eight bins on, workspaces past
128 MB): the first and the last rows of such fields, all columns (edges of the
64-vertex tiles, ragged ends, vector and scalar gathers), against the oracle on
the same rows, and the batched form with a field of another rule beside it."""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_18015_amd as cp
import workloads
from paper_2407_18015_amd import _lib as L

pytestmark = pytest.mark.gpu
HST = L.CP_HISTOGRAM


def field(H, W, nb, dtype, seed=3):
    p = workloads.random_params(HST, seed, H, W, nbins=nb, width=0.06)
    rng = np.random.default_rng(seed)
    up = [rng.normal(size=(H, W)) for _ in range(2)]
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")  # noqa: E731
    return dev(p), [dev(u) for u in up]


@pytest.mark.parametrize("H,W,nb,dtype", [(596, 607, 18, torch.float32), (596, 608, 18, torch.float32),
                                          (1030, 750, 8, torch.float32), (700, 832, 10, torch.float32),
                                          (500, 487, 13, torch.float64), (600, 642, 8, torch.float64)])
def test_row_sums_against_oracle(H, W, nb, dtype):
    p, up = field(H, W, nb, dtype)
    p[0, 2, 65] = float("nan")  # an invalid stencil beside a tile edge
    g = cp.backward(p, *up, cp.field_of(p, HST, nb)).cpu().numpy().astype(np.float64)
    for rows, keep in ((slice(0, 14), slice(0, 12)), (slice(H - 14, H), slice(2, 14))):
        crop = [t[..., rows, :].contiguous() for t in (p, *up)]  # below the rule's size: entries stored directly
        direct = cp.backward(*crop, cp.field_of(crop[0], HST, nb)).cpu().numpy()[:, keep]
        a = [t.cpu().numpy().astype(np.float64) for t in crop]
        ref, size = oracle.grad(HST, *a), oracle.grad(HST, *a, absolute=True)
        got, ref, size = g[:, rows][:, keep], ref[:, keep], size[:, keep]
        assert np.array_equal(np.isnan(got), np.isnan(direct))
        # the parity bound of the adjoint
        rel, s = (1e-5, 5e-7) if dtype == torch.float32 else (1e-10, 1e-13)
        assert np.nanmax(np.abs(got - ref) - (rel * (1 + np.abs(ref)) + s * size)) <= 0


def test_row_sums_batched_with_other_rules():
    fields, ps, ups, grads = [], [], [], []
    for H, W, nb in ((596, 607, 18), (40, 70, 19), (700, 832, 10), (33, 130, 3)):
        p, up = field(H, W, nb, torch.float32, seed=H)
        fields.append(cp.field_of(p, HST, nb))
        ps.append(p)
        ups.append(up)
        grads.append(torch.empty_like(p))
    cp.batched(fields, ps, gmin=[u[0] for u in ups], gmax=[u[1] for u in ups], grad=grads)
    for f, p, u, g in zip(fields, ps, ups, grads):
        assert torch.equal(g, cp.backward(p, *u, f))
