"""GPU parity of fp32 products through two fp16 terms per value, where the terms and their row scales can go wrong: rows that
end inside a split workgroup's registers or go beyond them, columns of very different magnitude, gradients that are tiny
beside others.  (Tiles and non-finite values: test_gpu_split.py.)

Tolerance.  A value keeps 23 bits, or 2^-40 of its row's largest one, and x2 y2 <= 2^-22 |x y| is left out: over a sum of
d <= 4128 products of std s that is at most sqrt(d) s 2^-21 as a random walk, 3e-5 of ONE product's size times sqrt(d) < 2e-6 for
the logits here (std 1).  The roundings of the fp32 sums (3 d / 32 <= 390, each 2^-24 of a partial sum below 5) come to 5e-6.
LOG = 2e-5, the bound of the other fp32 tests, for a log-probability, times sqrt(n) for a sum of n; a probability is then off by
2e-5 of itself, and so is a row of gradients that consists of nothing else: ROW = 3e-5 of the norm of that row.  Rows whose
terms cancel are off by more, on the fp32 instruction as well (the step that recomputes its logits takes that): half as much
again as there is allowed on top."""
import numpy as np
import pytest
import torch

import mtpc_inputs as mi
from oracle import backward as bw
from oracle import mtpc_oracle as oc
from gpu_util import make_head, takes_terms

pytestmark = pytest.mark.gpu

LOG, ROW = 2e-5, 3e-5


def prefix_error(inp):
    head = make_head(inp)
    assert takes_terms(head)
    logphi, logw, _ = oc._params(inp.family, inp.h, inp.W, inp.Wsum, None)
    want = oc.prefix_marginals_from(inp.family, logphi, logw, None, inp.targets)
    return np.abs(head.prefix_marginals(torch.from_numpy(inp.targets).cuda()).cpu().numpy() - want).max()


@pytest.mark.parametrize("d", [480, 512, 544, 4064, 4096, 4128])
@pytest.mark.parametrize("B,v", [(257, 33), (264, 40)])
def test_row_lengths(B, v, d):
    """Rows of one step of a split workgroup (512 columns) and next to it, and around those kept in registers (4096)."""
    assert prefix_error(mi.make_inputs("cp", B=B, d=d, n=8, r=11, v=v, dtype="f32", seed=d, h_scale=1.0)) < LOG * 8 ** 0.5


@pytest.mark.parametrize("power", [8, 12, 14, 16, 20, 40, 100])
@pytest.mark.parametrize("cols", [1, 40, 500])
def test_features_of_different_magnitude(power, cols):
    """`cols` features of h larger by 2^power, and W's smaller by as much: the logits are what they were.  (Rows of which too
    much is small beside their largest value are left to the fp32 instruction.)"""
    inp = mi.make_inputs("cp", B=257, d=512, n=8, r=11, v=33, dtype="f32", seed=power, h_scale=1.0)
    inp.h[:, :cols] *= 2.0 ** power
    inp.W[..., :cols] *= 2.0 ** -power
    inp.Wsum[:, :cols] *= 2.0 ** -power
    assert prefix_error(inp) < LOG * 8 ** 0.5


@pytest.mark.parametrize("family,B,d,n,r,v", [("ff", 300, 512, 3, 1, 33), ("cp", 513, 544, 4, 20, 40)])
def test_gradients_far_below_the_others(family, B, d, n, r, v):
    """Tokens that are never a target and next to impossible, positions with next to no weight, weights and features of many
    magnitudes: every row of dW and dh is right for its own size (forward pass with and without terms)."""
    rng = np.random.default_rng(B)
    inp = mi.make_inputs(family, B=B, d=d, n=n, r=r, v=v, dtype="f32", seed=B, h_scale=1.0)
    assert takes_terms(make_head(inp)) == (family == "cp")
    inp.h[:, 0] = 1.0
    inp.W[:, :, :, 0] = 0.0
    inp.W[:, :, v - 8:, 0] = -np.array([5, 9, 12, 15, 18, 20, 25, 30], np.float32)    # probabilities down to e^-30
    inp.targets[:] = rng.integers(0, v - 8, size=inp.targets.shape)
    inp.W[:, :, 3] *= 2.0 ** -9                          # a row of weights far below the others
    inp.h[:, 7] *= 2.0 ** 9                              # ... and a feature far above
    inp.W[..., 7] *= 2.0 ** -9
    if inp.Wsum is not None:
        inp.Wsum[:, 7] *= 2.0 ** -9
    coef = bw.loss_coefficients(0.8, np.ones((B, n), bool)) * 2.0 ** -rng.integers(0, 40, size=(B, 1))
    coef = coef.astype(np.float32)
    ref = bw.loss_and_gradients(family, inp.h, inp.W, inp.Wsum, inp.layers, inp.targets, coef)
    tg, cf = torch.from_numpy(inp.targets.astype(np.int32)).cuda(), torch.from_numpy(coef).cuda()
    out, plain = make_head(inp).loss_backward(tg, cf), make_head(inp).loss_backward(tg, cf, recompute=True)
    for k in ("dW", "dh"):
        size = np.linalg.norm(ref[k], axis=-1)
        assert (size > 0).all()
        worst = [(np.linalg.norm(o[k].cpu().numpy().astype(np.float64) - ref[k], axis=-1) / size).max() for o in (out, plain)]
        print(k, "worst row", worst)
        assert worst[0] < ROW + 1.5 * worst[1], (k, worst)
