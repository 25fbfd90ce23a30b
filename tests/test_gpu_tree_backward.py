"""GPU parity of the tree's reverse pass on the matrix pipes (shared layers of 16, 32 or 64 units) against the
float64 reverse-mode oracle: every depth of the tree, row counts that leave a workgroup partly or nearly empty,
one matrix for all nodes, and sizes that are left to the kernel with one wave per row (n = 32 at r = 32).
Tolerances: those of test_gpu_backward (the same check), but for dWsum.  Its entries are differences of the
posteriors of neighbouring prefixes, which for a deep tree nearly cancel: sum_j g_j softmax_j[z] - omega_z sum_j g_j.
A posterior is the exponential of a difference of logs of size |P| < 64, so it carries a relative error of up to
64 * 2^-23 = 8e-6, and an entry of dWsum one of up to 8e-6 * sum |g_j| * max softmax * |h| per position, twice (the
kernel with one wave per row shows the same errors: 1.5e-4 of the norm for one row, n = 16, r = 64, 6.6e-5 for forty)."""
import numpy as np
import pytest
import torch

from oracle import backward as bw
from gpu_util import make_head
from test_gpu_backward import check_grad, make_case

pytestmark = pytest.mark.gpu

CASES = [("btree", "f32", 33, 64, 2, 16, 20), ("btree", "f32", 16, 64, 4, 64, 33), ("btree", "f32", 17, 64, 8, 32, 33),
         ("btree", "f32", 1, 64, 16, 64, 24), ("btree", "bf16", 70, 64, 16, 64, 40), ("btree-shared", "f32", 31, 64, 8, 16, 40),
         ("btree", "f32", 18, 32, 32, 16, 12), ("btree", "f32", 6, 32, 32, 32, 12)]


@pytest.mark.parametrize("family,dtype,B,d,n,r,v", CASES)
def test_tree_reverse_pass(family, dtype, B, d, n, r, v):
    inp, targets, coef = make_case(family, dtype, B, d, n, r, v, seed=B + n + r)
    head = make_head(inp)
    args = torch.from_numpy(targets).cuda(), torch.from_numpy(coef.astype(np.float32)).cuda()
    out = head.loss_backward(*args)
    ref = bw.loss_and_gradients("btree", inp.h, inp.W, inp.Wsum, inp.layers if n > 2 else None, targets, coef.astype(np.float32))
    assert np.abs(out["loss"].cpu().numpy() - ref["loss"]).max() < 1e-4
    for k in ("dh", "dW", "dlayers"):
        if out[k] is not None and ref[k] is not None:
            check_grad(k, out[k], ref[k], dtype)
    g = np.abs(np.diff(np.concatenate([coef, np.zeros((B, 1))], axis=1), axis=1)).sum()
    bound = 2 * 8e-6 * g * np.abs(inp.h).max() + (2e-2 if dtype == "bf16" else 2e-5) * np.abs(ref["dWsum"]).max()
    assert np.abs(out["dWsum"].cpu().numpy() - ref["dWsum"]).max() <= bound
    again = head.loss_backward(*args)
    assert all(torch.equal(again[k], out[k]) for k in out if out[k] is not None)


def test_zero_weights_and_summed_out_windows():
    """-inf layer logits (weights of exactly zero) and windows whose variables are all summed out."""
    inp, targets, coef = make_case("btree", "f32", 40, 64, 8, 16, 33, seed=3)
    inp.layers[:, :, 3] = -np.inf
    targets[5] = -1
    head = make_head(inp)
    out = head.loss_backward(torch.from_numpy(targets).cuda(), torch.from_numpy(coef.astype(np.float32)).cuda())
    ref = bw.loss_and_gradients("btree", inp.h, inp.W, inp.Wsum, inp.layers, targets, coef.astype(np.float32))
    for k in ("dh", "dW", "dWsum"):
        check_grad(k, out[k], ref[k], "f32")
    fin = np.isfinite(ref["dlayers"])
    assert np.abs(out["dlayers"].cpu().numpy() - ref["dlayers"])[fin].max() < 2e-5 * np.abs(ref["dlayers"][fin]).max()
