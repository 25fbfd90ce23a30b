"""GPU parity of the training step's contraction over tokens (dh), whose operands are read along their rows: W and, in bf16, the
logit gradient as they lie in memory, transposed on the way out of LDS.

Sizes: rows of W that end inside a stage of 32 (with and without the rows of the sum units behind them), columns that end
inside a block of 64 or a tile of 256, positions that end inside a chunk of 32 or a tile, sums long enough to be split.  In bf16 most
small steps keep their transposes: the second test has the sizes that do not, and asks.

Tolerance: that of the other gradient tests (check_grad).  Against the plan that recomputes its logits and reads transposed
copies, dh sums the same bf16 products in the same order of stages, but the probabilities were formed from a
recomputed logit: a rounding step of the logit gradient here and there, 2^-9 of a term, as the bf16 tolerance has it.  (The
smallest vocabulary has two tokens: with one every gradient is 0, and a relative bound on it says nothing.)"""
import numpy as np
import pytest
import torch

import mtpc_inputs as mi
from oracle import backward as bw
from gpu_util import make_head, takes_row_operands
from test_gpu_backward import check_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("family,B,d,n,r,v", [("ff", 65, 32, 3, 1, 33), ("ff", 256, 64, 4, 1, 32), ("cp", 70, 96, 3, 5, 33), ("cp", 257, 288, 2, 7, 61),
                                              ("hmm", 300, 256, 5, 8, 100), ("btree", 129, 320, 4, 16, 257), ("cp", 600, 64, 8, 33, 31),
                                              ("hmm", 320, 544, 4, 16, 129), ("ff", 97, 512, 64, 1, 320), ("cp", 80, 32, 1, 3, 2)])
def test_dh_and_the_rest(family, B, d, n, r, v, dtype):
    inp = mi.make_inputs(family, B=B, d=d, n=n, r=r, v=v, dtype=dtype, seed=B + d, h_scale=1.0)
    coef = bw.loss_coefficients(0.8, np.random.default_rng(B).random((B, n)) > 0.15).astype(np.float32)
    tg, cf = torch.from_numpy(inp.targets.astype(np.int32)).cuda(), torch.from_numpy(coef).cuda()
    out, other = make_head(inp).loss_backward(tg, cf), make_head(inp).loss_backward(tg, cf, recompute=True)
    ref = bw.loss_and_gradients(family, inp.h, inp.W, inp.Wsum, inp.layers, inp.targets, coef)
    for k in ("dh", "dW", "dWsum", "dlayers"):
        if out[k] is not None:
            check_grad(k, out[k], ref[k], dtype)
            check_grad(k, other[k], ref[k], dtype)
    again = make_head(inp).loss_backward(tg, cf)
    assert all(torch.equal(again[k], out[k]) for k in out if out[k] is not None)


# one tile, 8 stages and a ninth of sum units; positions and columns beyond a tile; 6 tiles; 108 tiles whose sums are split in
# four, the last part 51 stages of W's own rows and two of the rows behind; the same where W ends with a stage; without
# sum units; no whole stage at all, and fewer gradients than the padding of their rows
@pytest.mark.parametrize("family,B,d,n,r,v", [("cp", 70, 96, 3, 5, 17), ("cp", 257, 288, 2, 3, 61), ("hmm", 300, 544, 3, 5, 27), ("cp", 600, 2080, 8, 33, 31),
                                              ("btree", 289, 3104, 4, 16, 129), ("ff", 97, 3616, 29, 1, 317), ("cp", 33, 32, 1, 2, 2)])
def test_bf16_steps_along_rows(family, B, d, n, r, v):
    assert takes_row_operands(make_head(mi.make_inputs(family, B=B, d=d, n=n, r=r, v=v, dtype="bf16", seed=B + d, h_scale=1.0)))
    test_dh_and_the_rest(family, B, d, n, r, v, "bf16")
