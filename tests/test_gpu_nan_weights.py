"""Root weights that are NaN (a Wsum that has diverged) beside input units that are sound: every score that they enter is NaN, in calls of
few rows and of many, whatever the number of units is rounded up to."""
import numpy as np
import pytest
import torch

import mtpc_inputs as mi
from gpu_util import make_head

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [3, 200, 300, 2100])
@pytest.mark.parametrize("r", [3, 5, 8, 20, 64])
@pytest.mark.parametrize("family", ["cp", "hmm"])
def test_scores(family, r, B):
    inp = mi.make_inputs(family, B=B, d=32, n=4, r=r, v=9, dtype="f32", seed=r, h_scale=1.0)
    inp.Wsum[0, 0] = np.nan
    head, x = make_head(inp), torch.from_numpy(inp.targets).cuda()
    table = torch.full((B, 4, r, 9), -2.0, dtype=torch.float32, device="cuda")
    for got in (head.prefix_marginals(x), head.loglik(x), head.table_scores(table, x, prefix=True), head.table_scores(table, x)):
        assert bool(torch.isnan(got).all())
