"""GPU parity of the fp32 products through three bf16 terms per value (the 256-position tiles) against the
same sums in 64 bits.

Tolerance.  The terms are exact and the six products kept leave out less than 2^-25 |x y|, so a logit of d
terms is off by the rounding of its fp32 sums, as on the fp32 matrix pipes: at most (6 d / 32 + d) 2^-24 sum |x y|
(worst case, every rounding the same way; d <= 1056 and sum |x y| < 60 here: 4e-3, seen 6e-6).  The bounds used are those
of the other fp32 tests: 1e-4 on log-probabilities, 2e-5 of the largest gradient entry.

The sizes have enough slabs (n r) for the 256-position tiles: fewer go to narrower ones (unembed_positions)."""
import numpy as np
import pytest
import torch

import mtpc_inputs as mi
from oracle import backward as bw
from oracle import mtpc_oracle as oc
from oracle import philox
from gpu_util import FP32_ABS, compare_drafts, make_head
from test_gpu_backward import check_grad

pytestmark = pytest.mark.gpu


# edges of the vocabulary and position tiles, one column block, an odd and an even number of them, rows of h apart
SIZES = [(65, 512, 3, 43, 33), (70, 544, 43, 3, 128), (256, 512, 8, 9, 129), (257, 512, 8, 8, 256), (300, 1056, 8, 8, 268),
         (129, 1024, 11, 8, 320), (65, 512, 43, 3, 192), (66, 512, 43, 3, 193), (80, 544, 43, 3, 272), (80, 544, 43, 3, 273),
         (260, 512, 8, 8, 265)]


@pytest.mark.parametrize("B,d,n,r,v", SIZES)
def test_evidence_table_and_draws(B, d, n, r, v):
    inp = mi.make_inputs("cp", B=B, d=d, n=n, r=r, v=v, dtype="f32", seed=B + v, h_scale=1.0)
    head = make_head(inp)
    logphi, logw, _ = oc._params("cp", inp.h, inp.W, inp.Wsum, None)
    want = oc.prefix_marginals_from("cp", logphi, logw, None, inp.targets)
    got = head.prefix_marginals(torch.from_numpy(inp.targets).cuda()).cpu().numpy()
    assert np.abs(got - want).max() < FP32_ABS
    table = torch.full((B, n, r, v), float("nan"), device="cuda")
    drafts, lat, scores = head.sample(2, seed=5, want_prefix=True, logphi=table)
    assert np.abs(table.cpu().numpy() - logphi).max() < FP32_ABS
    want = oc.prefix_marginals_from("cp", logphi, logw, None, drafts[:, 1].cpu().numpy())
    assert np.abs(scores[:, 1].cpu().numpy() - want).max() < FP32_ABS


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.4028235e38, -3.4e38, 1e-38])
def test_values_at_the_ends_of_the_range(value):
    """An infinite or NaN weight gives what fp32 sums give; the largest finite ones stay finite terms."""
    B, d, n, r, v = 65, 512, 3, 43, 40
    inp = mi.make_inputs("cp", B=B, d=d, n=n, r=r, v=v, dtype="f32", seed=9, h_scale=1.0)
    inp.h = np.abs(inp.h) + 0.5
    inp.W[0, 1, 7, 5] = value
    # (times 0 for the largest: the softmax of a logit of 1e37 is beyond fp32, with any product kernel)
    inp.h[:, 5] = 0.0 if value == 3.4028235e38 else 0.25
    logits = np.einsum("nrvd,bd->bnrv", inp.W.astype(np.float64), inp.h.astype(np.float64))
    m = logits.max(axis=-1, keepdims=True)
    m[np.isneginf(m)] = 0
    with np.errstate(invalid="ignore"):
        want = logits - m - np.log(np.exp(logits - m).sum(axis=-1, keepdims=True))
    got = make_head(inp)
    table = torch.empty(B, n, r, v, device="cuda")
    got.sample(1, seed=5, want_prefix=True, logphi=table)
    got = table.cpu().numpy().astype(np.float64)
    other = np.ones((B, n, r, v), bool)
    other[:, 0, 1] = False
    assert np.abs(got - want)[other].max() < 1e-4        # (|logits| up to 400 here)
    with np.errstate(invalid="ignore"):
        same = (got == want) | (np.isnan(got) & np.isnan(want)) | (np.abs(got - want) <= 1e-4 + 1e-6 * np.abs(want))
    # (a unit with a NaN logit has no distribution: all that its softmax promises is that this entry is NaN)
    assert (same if not np.isnan(value) else same[:, 0, 1, 7]).all()


@pytest.mark.parametrize("family,B,d,n,r,v", [("cp", 65, 96, 2, 3, 33), ("hmm", 300, 544, 3, 5, 129), ("ff", 257, 512, 3, 1, 268),
                                              ("btree", 97, 512, 4, 6, 320)])
def test_training_step(family, B, d, n, r, v):
    inp = mi.make_inputs(family, B=B, d=d, n=n, r=r, v=v, dtype="f32", seed=B, h_scale=1.0)
    coef = bw.loss_coefficients(0.8, np.random.default_rng(B).random((B, n)) > 0.15)
    head = make_head(inp)
    tg = torch.from_numpy(inp.targets.astype(np.int32)).cuda()
    out = head.loss_backward(tg, torch.from_numpy(coef.astype(np.float32)).cuda())
    ref = bw.loss_and_gradients(family, inp.h, inp.W, inp.Wsum, inp.layers, inp.targets, coef.astype(np.float32))
    for k in ("dh", "dW", "dWsum", "dlayers"):
        if out[k] is not None:
            check_grad(k, out[k], ref[k], "f32")
    again = head.loss_backward(tg, torch.from_numpy(coef.astype(np.float32)).cuda())
    assert all(torch.equal(again[k], out[k]) for k in out if out[k] is not None)


@pytest.mark.parametrize("v", [129, 192, 193, 257, 264, 265, 272, 273])
@pytest.mark.parametrize("B,S,r", [(70, 1, 43), (300, 3, 18)])
def test_bf16_vocabulary_tiles(v, B, S, r):
    """The row counts at which the 256-position tiles and the gathered draws change their tile (192, 272 with
    one wave a block short, 320): evidence, table, draws through buckets and in the kernel."""
    inp = mi.make_inputs("hmm", B=B, d=96, n=3, r=r, v=v, dtype="bf16", seed=v + B, h_scale=1.0)
    logphi, logw, lay = oc._params("hmm", inp.h, inp.W, inp.Wsum, inp.layers)
    head = make_head(inp)
    want = oc.prefix_marginals_from("hmm", logphi, logw, lay, inp.targets)
    assert np.abs(head.prefix_marginals(torch.from_numpy(inp.targets).cuda()).cpu().numpy() - want).max() < 2e-5
    table = torch.full((B, 3, r, v), float("nan"), device="cuda")
    head.sample(S, seed=3, logphi=table)
    assert np.abs(table.cpu().numpy() - logphi).max() < 2e-5
    u = philox.uniforms(B, S, 6, seed=3)
    od, ol, margin = oc.sample_from("hmm", logphi, logw, lay, u, with_margin=True)
    for prefix in (False, True):                     # through buckets; in the fused kernel where those do not pay
        gd, gl, _ = head.sample(S, seed=3, want_prefix=prefix)
        compare_drafts(gd, gl, od, ol, margin)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,d,n,r,v", [(33, 64, 2, 64, 33), (64, 96, 2, 65, 320), (65, 64, 2, 3, 130), (97, 96, 3, 1, 320),
                                       (250, 64, 4, 16, 256), (257, 128, 2, 25, 40), (257, 64, 2, 26, 40),
                                       (65, 96, 3, 65, 265), (128, 64, 3, 43, 130), (129, 64, 3, 43, 320), (300, 64, 2, 40, 272)])
def test_few_tiles(B, d, n, r, v, dtype):
    """Batches that need fewer than 256 positions to a tile, or leave CUs idle with them: several tiles of 32, 64 or
    128 (and the first sizes beyond)."""
    inp = mi.make_inputs("ff" if r == 1 else "cp", B=B, d=d, n=n, r=r, v=v, dtype=dtype, seed=B + v, h_scale=1.0)
    logphi, logw, _ = oc._params(inp.family, inp.h, inp.W, inp.Wsum, None)
    head = make_head(inp)
    want = oc.prefix_marginals_from(inp.family, logphi, logw, None, inp.targets)
    assert np.abs(head.prefix_marginals(torch.from_numpy(inp.targets).cuda()).cpu().numpy() - want).max() < FP32_ABS
    nl = 0 if r == 1 else 1
    u = philox.uniforms(B, 1, n + nl, seed=3)
    od, ol, margin = oc.sample_from(inp.family, logphi, logw, None, u, with_margin=True)
    table = torch.full((B, n, r, v), float("nan"), device="cuda")
    for kw in ({}, {"want_prefix": True}, {"logphi": table}):
        gd, gl, _ = head.sample(1, seed=3, **kw)
        compare_drafts(gd, gl, od, ol, margin)
    assert np.abs(table.cpu().numpy() - logphi).max() < FP32_ABS
