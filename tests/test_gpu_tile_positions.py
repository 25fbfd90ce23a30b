"""GPU parity of the passes over W whose tiles hold 192 or 128 positions because that saves rounds over the CUs: batches that
fill such a tile, end one short of it and one beyond it, with every number of vocabulary rows a tile can have.

132 slabs (n r) on 256 CUs: up to B = 192 one round of 192 positions as of 256 (192 are taken), up to 256 one of 256 only, up
to 384 two rounds of either and of 128 (128 are taken), up to 512 two of 256 and 192.

Tolerance.  A logit of standard deviation 1 is a sum of d <= 96 exact products in fp32: its roundings are below 96 2^-24 of its
terms' size, 1e-5 with those of the normalisation; a window sums n = 4 of them.  Probabilities and gradients: as in the other
tests of them."""
import numpy as np
import pytest
import torch

import mtpc_inputs as mi
from oracle import backward as bw
from oracle import mtpc_oracle as oc
from gpu_util import make_head, takes_terms
from test_gpu_backward import check_grad

pytestmark = pytest.mark.gpu

LOG = 2e-5


@pytest.mark.parametrize("v", [33, 128, 129, 192, 193, 257, 272, 273, 320])
@pytest.mark.parametrize("B", [129, 191, 192, 193, 300, 449])
def test_scores_and_table(B, v):
    inp = mi.make_inputs("cp", B=B, d=96, n=4, r=33, v=v, dtype="bf16", seed=B + v, h_scale=1.0)
    logphi, logw, _ = oc._params("cp", inp.h, inp.W, inp.Wsum, None)
    head = make_head(inp)
    got = head.prefix_marginals(torch.from_numpy(inp.targets).cuda()).cpu().numpy()
    assert np.abs(got - oc.prefix_marginals_from("cp", logphi, logw, None, inp.targets)).max() < LOG * 4
    uni = head.univariate_marginals().cpu().numpy()
    assert np.abs(uni - oc.univariate_marginals("cp", inp.h, inp.W, inp.Wsum, None)).max() < LOG * 4
    head.pack_W()                                       # the copy of W in 64-byte stages: the same products in the same order
    again = head.prefix_marginals(torch.from_numpy(inp.targets).cuda()).cpu().numpy()
    assert np.array_equal(again, got)


@pytest.mark.parametrize("v", [33, 100, 190, 268, 300])
@pytest.mark.parametrize("B", [257, 383, 384, 385])
def test_fp32_terms(B, v):
    """(136 slabs: two rounds of 192 positions as of 256 for all of these.)"""
    for d, terms in ((32, None), (512, True)):
        inp = mi.make_inputs("cp", B=B, d=d, n=8, r=17, v=v, dtype="f32", seed=B + v, h_scale=1.0)
        head = make_head(inp)
        assert terms is None or takes_terms(head) == terms
        logphi, logw, _ = oc._params("cp", inp.h, inp.W, inp.Wsum, None)
        got = head.prefix_marginals(torch.from_numpy(inp.targets).cuda()).cpu().numpy()
        assert np.abs(got - oc.prefix_marginals_from("cp", logphi, logw, None, inp.targets)).max() < LOG * 8 ** 0.5


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,d,v", [(129, 64, 33), (192, 96, 268), (300, 544, 61), (385, 512, 100)])
def test_training_step(B, d, v, dtype):
    inp = mi.make_inputs("cp", B=B, d=d, n=4, r=33, v=v, dtype=dtype, seed=B, h_scale=1.0)
    coef = bw.loss_coefficients(0.8, np.random.default_rng(B).random((B, 4)) > 0.15).astype(np.float32)
    out = make_head(inp).loss_backward(torch.from_numpy(inp.targets.astype(np.int32)).cuda(), torch.from_numpy(coef).cuda())
    ref = bw.loss_and_gradients("cp", inp.h, inp.W, inp.Wsum, inp.layers, inp.targets, coef)
    for k in ("dh", "dW", "dWsum"):
        check_grad(k, out[k], ref[k], dtype)
