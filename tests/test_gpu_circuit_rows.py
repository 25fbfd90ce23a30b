"""GPU parity of the circuits of few rows (a workgroup to a row): every width a product can have, windows of one token to 64, layers shared
and of every position, evidence from rows and from a kept table, rows on both sides of what the narrower form and the other kernels take,
and evidence so far apart that the linear values of the HMM's chain do not hold it.

Tolerances: fp32 inputs as in the other parity tests; the extreme evidence sums to magnitudes of up to 3e3, where an fp32 result
has 2^-23 of its value, and the units' logarithms before it as much of theirs: 4 2^-23 of the value."""
import numpy as np
import pytest
import torch

import mtpc_inputs as mi
from oracle import mtpc_oracle as oc
from gpu_util import make_head, tol_check

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (2, 3), (4, 8), (16, 9), (8, 16), (16, 17), (64, 2), (16, 32), (4, 33), (16, 50), (8, 64), (16, 64), (32, 30)]


@pytest.mark.parametrize("B", [3, 256, 257, 300])
@pytest.mark.parametrize("n,r", SHAPES)
@pytest.mark.parametrize("family", ["cp", "hmm", "btree"])
def test_scores(family, n, r, B):
    n = max(n, 2) if family == "btree" else n              # (a tree has two leaves at least)
    inp = mi.make_inputs(family, B=B, d=32, n=n, r=r, v=5, dtype="f32", seed=n + r, h_scale=1.0)
    logphi, logw, lay = oc._params(family, inp.h, inp.W, inp.Wsum, inp.layers)
    x = inp.targets.astype(np.int32).copy()
    x[0, 0], x[1, n // 2], x[2, -1] = -1, 5, -1             # summed out, no such id, summed out
    want = oc.prefix_marginals_from(family, logphi, logw, lay, x)
    head, tx = make_head(inp), torch.from_numpy(x).cuda()
    got = head.prefix_marginals(tx)
    tol_check(got.cpu().numpy(), want, "f32", "prefix")
    assert torch.equal(head.loglik(tx).nan_to_num(1.0), got[:, -1].nan_to_num(1.0))
    table = torch.from_numpy(logphi.astype(np.float32)).cuda()
    two = torch.stack([tx, tx.flip(0)], dim=1).contiguous()
    kept = head.table_scores(table, two, prefix=True).cpu().numpy()
    tol_check(kept[:, 0], want, "f32", "from the table")


@pytest.mark.parametrize("n,r", [(4, 5), (16, 16), (8, 40), (8, 64)])
@pytest.mark.parametrize("family", ["hmm", "btree"])
def test_layers_of_every_position(family, n, r):
    inp = mi.make_inputs(family, B=20, d=32, n=n, r=r, v=5, dtype="f32", seed=n + r, h_scale=1.0)
    lay = np.random.default_rng(1).standard_normal((20,) + inp.layers.shape)
    logphi, logw, ll = oc._params(family, inp.h, inp.W, inp.Wsum, lay)
    got = make_head(inp, layers=lay).prefix_marginals(torch.from_numpy(inp.targets).cuda()).cpu().numpy()
    tol_check(got, oc.prefix_marginals_from(family, logphi, logw, ll, inp.targets), "f32", family)


@pytest.mark.parametrize("r", [4, 16, 32, 64])
@pytest.mark.parametrize("family", ["cp", "hmm", "btree"])
def test_evidence_far_apart(family, r):
    n, B, v = 8, 40, 3
    inp = mi.make_inputs(family, B=B, d=32, n=n, r=r, v=v, dtype="f32", seed=r, h_scale=1.0)
    rng = np.random.default_rng(r)
    logphi = np.where(rng.random((B, n, r, v)) < 0.5, -rng.uniform(0, 400, (B, n, r, v)), -rng.uniform(0, 3, (B, n, r, v)))
    logphi[0] = -np.inf                                     # nothing left at all
    logphi[1, n // 2] = -np.inf
    lay = None if inp.layers is None else rng.uniform(-20, 20, inp.layers.shape)
    _, logw, ll = oc._params(family, inp.h, inp.W, inp.Wsum, lay)
    want = oc.prefix_marginals_from(family, logphi.astype(np.float32).astype(np.float64), logw, ll, inp.targets)
    table = torch.from_numpy(logphi.astype(np.float32)).cuda()
    got = make_head(inp, layers=lay).table_scores(table, torch.from_numpy(inp.targets).cuda()[:, None].contiguous(), prefix=True)
    got = got.cpu().numpy()[:, 0].astype(np.float64)
    assert np.array_equal(np.isneginf(got), np.isneginf(want))
    ok = np.isfinite(want)
    assert np.all(np.abs(got - want)[ok] <= 1e-4 + 4 * 2.0 ** -23 * np.abs(want[ok]))


@pytest.mark.parametrize("B", [1, 3, 17, 255])
@pytest.mark.parametrize("n,r", [(16, 60), (32, 40), (16, 64), (64, 32)])
def test_few_rows_of_trees_whose_layers_do_not_fit(n, r, B):
    inp = mi.make_inputs("btree", B=B, d=32, n=n, r=r, v=5, dtype="f32", seed=n + r, h_scale=1.0)
    logphi, logw, lay = oc._params("btree", inp.h, inp.W, inp.Wsum, inp.layers)
    x = inp.targets.astype(np.int32).copy()
    x[0, 0], x[-1, -1] = -1, 5                              # summed out, no such id
    head, tx = make_head(inp), torch.from_numpy(x).cuda()
    got = head.prefix_marginals(tx)
    tol_check(got.cpu().numpy(), oc.prefix_marginals_from("btree", logphi, logw, lay, x), "f32", "prefix")
    tol_check(head.loglik(tx).cpu().numpy(), got[:, -1].cpu().numpy(), "f32", "log-likelihood")
