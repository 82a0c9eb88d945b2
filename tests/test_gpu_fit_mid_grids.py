"""FP32 fits on both sides of the grid sizes that test for equal members by
comparisons instead of by the sum of squares: the fused fit, which uses the sum
throughout, gives the same bits, degenerate and NaN members among them."""
import pytest
import torch

import paper_2407_18015_amd as cp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(640, 1024), (641, 1024), (1024, 1024), (1152, 1024), (1153, 1024)])
@pytest.mark.parametrize("M", [2, 6, 9])
def test_equal_members(shape, M):
    torch.manual_seed(M)
    m = torch.randn(M, *shape, device="cuda")
    m[:, 1, 1] = 3.0
    m[:, 2, 1:9] = 0.0
    m[M - 1, 2, 3] = 1.4e-45
    m[:, 3, 4] = 4.0
    m[1, 3, 4] = float("nan")  # among equal members
    m[0, 5, 6] = float("nan")
    m[1, 7, 8] = float("inf")
    p, _, _ = cp.fit_forward(m, "epanechnikov")
    q = cp.fit(m, "epanechnikov")
    assert torch.equal(p.view(torch.int32), q.view(torch.int32))
    assert q[1, 1, 1] > 0 and q[1, 2, 3] != q[1, 2, 4]
    g = cp.fit(m, "gaussian")
    assert torch.equal(g[0].view(torch.int32), q[0].view(torch.int32))
