"""Monte Carlo forward on both sides of the sample count from which the generator's
keys sit in vector registers, one and two vertices per wave, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_18015_amd as cp
import workloads
from paper_2407_18015_amd import _lib as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns", [255, 256, 257])
@pytest.mark.parametrize("H,W", [(1, 2), (9, 7), (91, 91)])
def test_keys(H, W, ns):
    mem = workloads.correlated_ensemble(12, max(H, 8), max(W, 8))[:, :H, :W]
    params = cp.fit(torch.as_tensor(np.ascontiguousarray(mem), dtype=torch.float32, device="cuda"), "mvg")
    idx = np.arange(H * W) if H * W < 200 else np.arange(0, H * W, 211)
    ref, amb = oracle.mvg_forward_at(params.cpu().numpy(), idx, ns, 79, 7)
    for est, cols in ((L.CP_MC_CONDITIONAL, (2, 3)), (L.CP_MC_HIT, (0, 1))):
        f = cp.Field(H, W, L.CP_MVGAUSS, torch.float32, nsamples=ns, seed=79, field_id=7, estimator=est)
        for k, out in enumerate(cp.forward(params, f)):
            got, want = out.cpu().numpy().ravel()[idx].astype(np.float64), ref[:, cols[k]]
            if est == L.CP_MC_HIT:  # whole hits, equal but for the oracle's near-ties
                assert np.all(np.abs(np.rint(got * ns) - np.rint(want * ns)) <= amb[:, k])
            else:  # the parity bound of the estimator
                assert np.all(np.abs(got - want) <= 1e-6)
