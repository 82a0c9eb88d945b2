"""The FP32 adjoint's tile shapes (small, middle and large grids): a vertex's
gradient does not depend on the shape, so crops of a large field, which take the
smaller tiles, give its bits away from their own edges."""
import pytest
import torch

import paper_2407_18015_amd as cp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model", ["uniform", "epanechnikov", "gaussian"])
def test_crops_equal_the_whole(model):
    torch.manual_seed(5)
    H, W = 1231, 1277  # 42 x 43 tiles of 30 x 30 outputs
    p = torch.empty(2, H, W, device="cuda")
    p[0] = torch.rand(H, W, device="cuda")
    p[1] = 0.1 + torch.rand(H, W, device="cuda")
    if model == "uniform":
        p[1] += p[0]
    g = [torch.randn(H, W, device="cuda") for _ in range(2)]
    whole = cp.backward(p, *g, cp.field_of(p, model))
    # one tile and less, ragged, either side of 448 and 960 tiles
    for y0, x0, h, w in [(0, 0, 3, 5), (40, 30, 14, 15), (100, 77, 31, 61), (5, 9, 630, 630), (5, 9, 631, 630),
                         (3, 1, 929, 931), (200, 300, 931, 929), (0, 0, 1229, 1121)]:
        crop = [t[..., y0:y0 + h, x0:x0 + w].contiguous() for t in (p, *g)]
        got = cp.backward(*crop, cp.field_of(crop[0], model))
        a, b = got[:, 2:-2, 2:-2], whole[:, y0:y0 + h, x0:x0 + w][:, 2:-2, 2:-2]
        assert torch.equal(a, b), (y0, x0, h, w)
