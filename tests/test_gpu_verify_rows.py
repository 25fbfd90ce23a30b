"""GPU parity of the verification that keeps a position's layers in LDS: every width of its products up to 64 units, windows of one
token to 64, layers shared by all positions, one layer for all steps and nodes, layers of every position - as logits, which it normalises
itself, and computed from h -, batches on both sides of where a position's sum units are its own and of what takes another kernel, and
drafts that are rejected at the first, a middle and the last position, or not at all.

The verifier accepts what comes before the rejection for certain and gives the rejected token nothing, so that every row's length is given.
Tokens are compared where the final uniform is 2e-5 or more from a step (as in test_gpu_speculative)."""
import numpy as np
import pytest
import torch

import mtpc_inputs as mi
from oracle import mtpc_oracle as oc
from oracle import philox
from oracle import speculative as sp

from gpu_util import make_head, oracle_params

pytestmark = pytest.mark.gpu


def check(family, B, n, r, v, layers, dtype="f32", d=64):
    inp = mi.make_inputs(family, B=B, d=d, n=n, r=r, v=v, dtype=dtype, seed=B + n + r, h_scale=1.0,
                         layer_count=1 if layers == "one" else None, contextual=layers == "from h", logit_gain=2.0)
    rng = np.random.default_rng(n + r)
    lay = None
    if layers == "of every position":
        lay = rng.standard_normal((B,) + inp.layers.shape).astype(np.float32)
        logphi, logw, logT = oc._params(family, inp.h, inp.W, inp.Wsum, lay)
    else:
        logphi, logw, logT = oracle_params(inp)
    logphi = logphi.astype(np.float32).astype(np.float64)
    drafts = inp.targets
    where = np.array([0, n // 2, n - 1, n])[np.arange(B) % 4]
    p = rng.dirichlet(np.full(v, 0.5), size=(B, n + 1))
    for b, j in enumerate(where):
        p[b, :j] = 0.0
        p[b, np.arange(j), drafts[b, :j]] = 1.0
        if j < n:
            p[b, j, drafts[b, j]] = 0.0
            p[b, j] /= p[b, j].sum()
    u = philox.verify_uniforms(B, n + 1, 5, 2)
    want_acc, want_tok, margin = sp.speculative_verify(family, logphi, logw, logT, drafts, p, u)
    assert np.array_equal(want_acc, where)
    P = oc.prefix_marginals_from(family, logphi, logw, logT, drafts)
    acc, tok = make_head(inp, layers=lay).verify(torch.from_numpy(drafts).cuda(), torch.from_numpy(p.astype(np.float32)).cuda(),
                                                 prefix_logq=torch.from_numpy(P.astype(np.float32)).cuda(),
                                                 logphi=torch.from_numpy(logphi.astype(np.float32)).cuda(), seed=5, offset=2)
    assert np.array_equal(acc.cpu().numpy(), where)
    safe = margin >= 2e-5
    assert safe.sum() >= 0.9 * B
    assert np.array_equal(tok.cpu().numpy()[safe], want_tok[safe])


@pytest.mark.parametrize("n,r", [(1, 64), (4, 1), (8, 8), (16, 9), (16, 16), (16, 17), (16, 32), (16, 33), (8, 50), (8, 64), (64, 5), (32, 30),
                                 (16, 64)])                 # (the last: layers that do not fit, beside a CP that has none)
@pytest.mark.parametrize("family", ["cp", "hmm", "btree"])
def test_units_and_windows(family, n, r):
    check(family, 22, max(n, 2) if family == "btree" else n, r, 37, "shared")


@pytest.mark.parametrize("r", [7, 32, 64])
@pytest.mark.parametrize("layers", ["one", "of every position", "from h"])
@pytest.mark.parametrize("family", ["hmm", "btree"])
def test_layers(family, layers, r):
    check(family, 21, 8, r, 33, layers)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B", [1, 128, 129, 256, 257])
@pytest.mark.parametrize("family", ["ff", "cp", "hmm", "btree"])
def test_batches(family, B, dtype):
    check(family, B, 8, 1 if family == "ff" else 24, 320, "shared", dtype=dtype, d=96)
