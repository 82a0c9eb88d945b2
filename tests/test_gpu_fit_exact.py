"""The fit's shared divisors: quotients by M and by a vertex's range are correctly rounded.

Members are whole numbers, so the mean's sums are exact and numpy's IEEE division
gives the parameters; the histogram's bins follow numpy's division bit for bit."""
import numpy as np
import pytest
import torch

import paper_2407_18015_amd as cp

pytestmark = pytest.mark.gpu

COUNTS = [2, 3, 7, 9, 17, 33, 41]
TYPES = [(torch.float32, np.float32), (torch.float64, np.float64)]


def _members(M, H, W, nt, scale):
    m = np.random.default_rng(M * 7 + H).integers(-1000, 1000, (M, H, W)).astype(nt)
    m[:, 1, 1] = 5          # all equal: degenerate
    m[:, 2, 2] = 0
    m[0, 2, 3] = np.nan     # a NaN first member: degenerate
    m[1, 3, 3] = np.nan     # a NaN among members that differ
    m[:, 3, 4] = 4
    m[1, 3, 4] = np.nan     # a NaN among equal members
    return m * nt(scale)


@pytest.mark.parametrize("dt,nt", TYPES)
@pytest.mark.parametrize("M", COUNTS)
@pytest.mark.parametrize("W", [8, 7])  # by 16-byte groups, one by one
def test_epanechnikov_quotients(dt, nt, M, W):
    m = _members(M, 5, W, nt, 1)
    p = cp.fit(torch.from_numpy(m).cuda(), "epanechnikov").cpu().numpy()
    x = m.astype(np.float64)
    d = x - x[0]
    s1, s2 = d.sum(0), (d * d).sum(0)
    mean = x[0] + s1 / M
    with np.errstate(invalid="ignore"):
        ss = np.maximum(s2 - s1 * s1 / M, 0.0)
    ok = np.isfinite(mean) & (d != 0).any(0)
    assert np.array_equal(p[0][np.isfinite(mean)], mean[np.isfinite(mean)].astype(nt))
    w = 1.06 * M ** -0.2 * np.sqrt(ss / (M - 1))
    # the scale's own few roundings in 64 bits, and the result's
    assert np.allclose(p[1][ok], w[ok], rtol=16 * 2.0**-53 + np.finfo(nt).eps, atol=0)
    # a vertex of equal members keeps the degenerate width, as does a NaN first one
    q = cp.fit(torch.from_numpy(m[:, :, ::-1].copy()).cuda(), "epanechnikov").cpu().numpy()[:, :, ::-1]
    assert np.array_equal(p, q, equal_nan=True)
    assert np.isnan(p[0][2, 3]) and np.isnan(p[0][3, 3]) and p[1][1, 1] < p[1][ok].min()


@pytest.mark.parametrize("dt,nt", TYPES)
@pytest.mark.parametrize("M", COUNTS)
@pytest.mark.parametrize("scale", [1.0, 1e-36, 1e33, 0.1])  # ranges that divide in FP32, a rounded one
def test_histogram_bins(dt, nt, M, scale):
    m = _members(M, 40, 67, nt, scale)
    for nb in (1, 3, 10):
        p = cp.fit(torch.from_numpy(m).cuda(), "histogram", nbins=nb).cpu().numpy()
        good = np.isfinite(m).all(0) & (m.min(0) < m.max(0))
        lo, hi = m.min(0)[good], m.max(0)[good]
        assert np.array_equal(p[0][good], lo) and np.array_equal(p[1][good], hi)
        j = np.clip((((m[:, good] - lo) / (hi - lo)) * nt(nb)).astype(np.int64), 0, nb - 1)
        for b in range(nb):
            assert np.array_equal(p[2 + b][good], ((j == b).sum(0).astype(nt) / nt(M)))


@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
@pytest.mark.parametrize("model", ["uniform", "epanechnikov"])
@pytest.mark.parametrize("shape", [(5, 8), (9, 132), (13, 64), (700, 800), (1600, 2304)])
# (both tile heights, remainders, the fit's three loops)
def test_fused_fit_is_the_fit(dt, model, shape):
    for M in (1, 2, 7, 9, 20) if shape[0] < 100 else (9,):
        if M == 1 and model == "epanechnikov":
            continue
        torch.manual_seed(M)
        m = torch.randn(M, *shape, device="cuda", dtype=dt)
        m[:, 1, 1] = 3.0
        m[M // 2, 2, 2] = float("nan")
        p, _, _ = cp.fit_forward(m, model)
        assert torch.equal(p.nan_to_num(7.5), cp.fit(m, model).nan_to_num(7.5))
