"""GPU parity of the HMM's chain where its values lie far apart: root weights up to 120 nats apart with a first observation that
opposes them, evidence that takes units 80 nats down and brings them up again, with layers that hardly mix the units.  Scores of few rows
(a workgroup to a row) and of many, and verifications of few and of many positions.

Tolerances: fp32 evidence and weights of magnitudes up to 200, whose sums are rounded once a step (2^-17 at the most), and 4 2^-23 of the
result's own value; a drawn token is compared where its uniform is 2e-4 or more from a step."""
import numpy as np
import pytest
import torch

import mtpc_inputs as mi
from oracle import mtpc_oracle as oc
from oracle import philox
from oracle import speculative as sp

from gpu_util import make_head

pytestmark = pytest.mark.gpu

SIZES = [(1, 5), (3, 2), (8, 7), (8, 16), (16, 30), (4, 33), (8, 64)]


def far_apart(B, n, r, v, seed):
    """Inputs of an HMM, tokens and a table whose evidence at them sets the forward message of every step: at random up to 80 nats
    below its largest unit."""
    inp = mi.make_inputs("hmm", B=B, d=32, n=n, r=r, v=v, dtype="f32", seed=seed, h_scale=1.0)
    rng = np.random.default_rng(seed)
    inp.h[:], inp.Wsum[:] = 0.0, 0.0
    inp.h[:, 0], inp.Wsum[:, 0] = 1.0, rng.uniform(-120, 0, r)
    eye = np.eye(r, dtype=bool)[None]
    inp.layers[:] = np.where(eye, 0.0, rng.uniform(-85, -70, inp.layers.shape))
    logw, logT = oc.sum_unit(inp.h, inp.Wsum), oc.sum_layers(inp.layers)
    logphi = rng.uniform(-5, -1, (B, n, r, v)).astype(np.float32)
    x = inp.targets
    predicted = logw
    for i in range(n):
        e = rng.uniform(-80, 0, (B, r)) - predicted
        e = (e - e.max(axis=1, keepdims=True) - 1.0).astype(np.float32)
        np.put_along_axis(logphi[:, i], x[:, i, None, None].repeat(r, axis=1), e[:, :, None], axis=2)
        if i + 1 < n:
            predicted = oc.logsumexp((predicted + e)[:, :, None] + logT[i][None], axis=1)
    return inp, logphi, logw, logT


@pytest.mark.parametrize("n,r", SIZES)
def test_scores(n, r):
    B = 40
    inp, logphi, logw, logT = far_apart(B, n, r, 3, seed=n + r)
    want = oc.prefix_marginals_from("hmm", logphi.astype(np.float64), logw, logT, inp.targets)
    head, table = make_head(inp), torch.from_numpy(logphi).cuda()
    for T in (1, 52):                                       # 40 rows; 2080, too many for a workgroup to each
        x = torch.from_numpy(inp.targets).cuda()[:, None].expand(B, T, n).contiguous()
        got = head.table_scores(table, x, prefix=True).cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - want[:, None]) <= 1e-4 + 4 * 2.0 ** -23 * np.abs(want[:, None])), T
        joint = head.table_scores(table, x).cpu().numpy()
        assert np.array_equal(joint, got[:, :, -1].astype(np.float32))


@pytest.mark.parametrize("B", [48, 130, 300])
@pytest.mark.parametrize("n,r", SIZES)
def test_verification(n, r, B):
    v = 40
    inp, logphi, logw, logT = far_apart(B, n, r, v, seed=n + r)
    rng = np.random.default_rng(B)
    p = np.zeros((B, n + 1, v))
    drafts = inp.targets
    for b in range(B):
        j = b % (n + 1)                                     # accepted before, rejected here
        p[b, np.arange(n), drafts[b]] = 1.0
        p[b, j] = rng.dirichlet(np.full(v, 0.3))
        if j < n:
            p[b, j, drafts[b, j]] = 0.0
            p[b, j] /= p[b, j].sum()
            logphi[b, j] = np.log(rng.dirichlet(np.full(v, 0.3), size=r) + 1e-6)
    phi = logphi.astype(np.float64)
    u = philox.verify_uniforms(B, n + 1, 7, 1)
    want_acc, want_tok, margin = sp.speculative_verify("hmm", phi, logw, logT, drafts, p, u)
    assert np.array_equal(want_acc, np.arange(B) % (n + 1))
    P = oc.prefix_marginals_from("hmm", phi, logw, logT, drafts)
    acc, tok = make_head(inp).verify(torch.from_numpy(drafts).cuda(), torch.from_numpy(p.astype(np.float32)).cuda(),
                                     prefix_logq=torch.from_numpy(P.astype(np.float32)).cuda(), logphi=torch.from_numpy(logphi).cuda(),
                                     seed=7, offset=1)
    assert np.array_equal(acc.cpu().numpy(), want_acc)
    safe = margin >= 2e-4
    assert safe.sum() >= 0.9 * B
    assert np.array_equal(tok.cpu().numpy()[safe], want_tok[safe])

@pytest.mark.parametrize("n,r", [(1, 8), (2, 32), (3, 32), (8, 16), (16, 32)])
def test_scores_carry_one_rounding(n, r):
    """Evidence as a byte model has it.  The result's own rounding is 2^-24 of it at the most, 3.4e-8 in the mean square; the steps before
    it (linear values, errors of some 2^-24 each, in a magnitude of 5 a step) add less than that."""
    B, v = 235, 3
    inp = mi.make_inputs("hmm", B=B, d=32, n=n, r=r, v=v, dtype="f32", seed=n + r, h_scale=1.0)
    inp.Wsum[:] = 0.0                                       # (weights 1 / r: none of their error is in what is measured)
    logphi = (np.random.default_rng(r).standard_normal((B, n, r, v)) - 5.5).astype(np.float32)
    logw, logT = oc.sum_unit(inp.h, inp.Wsum), oc.sum_layers(inp.layers)
    want = oc.prefix_marginals_from("hmm", logphi.astype(np.float64), logw, logT, inp.targets)
    got = make_head(inp).table_scores(torch.from_numpy(logphi).cuda(), torch.from_numpy(inp.targets).cuda()[:, None].contiguous(), prefix=True)
    rel = (got.cpu().numpy()[:, 0].astype(np.float64) - want) / want
    print(f"n={n} r={r}: relative error rms {np.sqrt(np.mean(rel ** 2)):.2e}, max {np.abs(rel).max():.2e}")
    assert np.sqrt(np.mean(rel ** 2)) <= 6e-8
