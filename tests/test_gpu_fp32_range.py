"""GPU parity of fp32 scoring and training where one row, column or position is far larger or smaller than the others: the
products through two fp16 terms per value take out one scale per row, so operands that hold values too far apart have to be seen
and left to products that hold every value whole.

Every row and every column of a gradient is compared by itself, relative to its own norm: an error that hides behind a larger
neighbour counts.  Tolerance, as for gradients far below the others (test_gpu_fp16_terms.py): ROW = 3e-5 of the norm, and half
as much again as the step that recomputes its logits, on the fp32 instruction, is off on the same inputs."""
import numpy as np
import pytest
import torch

import mtpc_inputs as mi
from oracle import backward as bw
from oracle import mtpc_oracle as oc
from gpu_util import make_head, takes_terms
from test_gpu_split import without_planes

pytestmark = pytest.mark.gpu

LOG, ROW = 2e-5, 3e-5


def outlier(inp, coef, power, feature=None, weight=0.0):
    """Position 100 larger by 2^power (one feature, which no logit sees, or all) with `weight` of its gradient left."""
    if feature is None:
        inp.h[100] *= 2.0 ** power
    else:
        inp.h[100, feature] = 2.0 ** power
        inp.W[..., feature] = 0.0
        if inp.Wsum is not None:
            inp.Wsum[:, feature] = 0.0
    coef[100] *= weight


def zero_token(inp, coef, gain):
    inp.W *= gain
    inp.W[:, :, 3] = 0.0


def zero_sum_units(inp, coef, gain):
    inp.W *= gain
    if inp.Wsum is not None:
        inp.Wsum[:] = 0.0


def impossible_token(inp, coef, power):
    """A token whose weights are 2^power and whose probability is 0."""
    inp.h[:, 0] = 1.0
    inp.W[:, :, -1] = 0.0
    inp.W[:, :, -1, 0] = -2.0 ** power
    inp.targets[:] %= inp.v - 1


def weak_column(inp, coef, power):
    inp.W[..., 7] *= 2.0 ** -power
    if inp.Wsum is not None:
        inp.Wsum[:, 7] *= 2.0 ** -power


def small_positions(inp, coef, power):
    """A few positions far below the others in all features, which alone have a weight to speak of."""
    inp.h[40:44] *= 2.0 ** -power
    rest = np.ones(inp.B, bool)
    rest[40:44] = False
    coef[rest] *= 2.0 ** -power


def faint_positions(inp, coef, power):
    """A few positions whose weight is far below the others', and a feature that only they have."""
    inp.h[:40, 7] = inp.h[44:, 7] = 0.0
    coef[40:44] *= 2.0 ** -power


def no_features(inp, coef):
    """A position without features and a feature without values."""
    inp.h[100] = 0.0
    coef[100] *= 2.0 ** 20
    inp.h[:, 7] = 0.0


def no_weights(inp, coef, sums):
    inp.W[:] = 0.0
    if sums and inp.Wsum is not None:
        inp.Wsum[:] = 0.0


def tiny_weights(inp, coef, power):
    inp.W *= 2.0 ** -power


CASES = {
    "masked position 2^20": (outlier, 20), "masked feature 2^20": (outlier, 20, 7), "masked feature 2^28": (outlier, 28, 7),
    "masked feature 2^90": (outlier, 90, 7), "weak feature 2^28": (outlier, 28, 7, 2.0 ** -28), "feature 2^28": (outlier, 28, 7, 1.0),
    "feature 2^14": (outlier, 14, 7, 1.0), "zero token": (zero_token, 1.0), "zero token, small W": (zero_token, 2.0 ** -8),
    "zero token, confident": (zero_token, 3.0), "zero sum units": (zero_sum_units, 1.0), "zero sum units, confident": (zero_sum_units, 3.0),
    "zero sum units, small W": (zero_sum_units, 2.0 ** -8), "impossible token 2^12": (impossible_token, 12),
    "impossible token 2^24": (impossible_token, 24), "column 2^-14": (weak_column, 14), "column 2^-20": (weak_column, 20), "column 2^-28": (weak_column, 28),
    "small positions 2^-12": (small_positions, 12), "small positions 2^-20": (small_positions, 20), "small positions 2^-26": (small_positions, 26),
    "faint positions 2^-12": (faint_positions, 12), "faint positions 2^-20": (faint_positions, 20), "faint positions 2^-32": (faint_positions, 32),
    "no features": (no_features,), "no weights": (no_weights, False), "no weights at all": (no_weights, True), "tiny weights": (tiny_weights, 60),
}


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("family,B,d,n,r,v", [("cp", 257, 512, 8, 11, 33), ("ff", 300, 544, 3, 1, 33)])
def test_every_row_and_column_of_a_gradient(family, B, d, n, r, v, case):
    """(Forward pass with and without terms.)"""
    inp = mi.make_inputs(family, B=B, d=d, n=n, r=r, v=v, dtype="f32", seed=B, h_scale=1.0)
    coef = bw.loss_coefficients(0.8, np.random.default_rng(B).random((B, n)) > 0.15).astype(np.float32)
    CASES[case][0](inp, coef, *CASES[case][1:])
    assert takes_terms(make_head(inp)) == (family == "cp")
    ref = bw.loss_and_gradients(family, inp.h, inp.W, inp.Wsum, inp.layers, inp.targets, coef)
    tg, cf = torch.from_numpy(inp.targets.astype(np.int32)).cuda(), torch.from_numpy(coef).cuda()
    out, plain = make_head(inp).loss_backward(tg, cf), make_head(inp).loss_backward(tg, cf, recompute=True)
    bad = []
    for k in ("dW", "dh"):
        want = ref[k].reshape(-1, d)
        for axis, what in ((1, "row"), (0, "column")):
            size = np.linalg.norm(want, axis=axis)
            off = [np.linalg.norm(o[k].cpu().numpy().astype(np.float64).reshape(-1, d) - want, axis=axis) for o in (out, plain)]
            seen = size > 2.0 ** -100 * size.max()
            if size.max() < 1e-12:                       # (nothing but roundings of zero)
                assert all((o < 1e-6).all() for o in off)
                continue
            assert all(np.isfinite(o).all() and (o[~seen] <= size.max() * 2.0 ** -24).all() for o in off), (k, what)
            worst = [(o[seen] / size[seen]).max() for o in off]
            print(case, k, what, "worst %.2g, on the fp32 instruction %.2g" % tuple(worst))
            if not worst[0] < ROW + 1.5 * worst[1]:
                bad.append((k, what, worst))
    assert not bad


@pytest.mark.parametrize("kept", [4, 20, 31])
@pytest.mark.parametrize("power", [20, 30])
def test_sparse_rows_with_an_outlier(kept, power):
    """Rows of h with a few values other than 0 (fewer than one in 16) and one far above them, which W does not see."""
    inp = mi.make_inputs("cp", B=257, d=512, n=8, r=11, v=33, dtype="f32", seed=power, h_scale=1.0)
    rng = np.random.default_rng(kept)
    for b in range(0, inp.B, 3):
        off = rng.permutation(np.arange(1, inp.d))[kept:]
        inp.h[b, off] = 0.0
        inp.h[b, 0] = 2.0 ** power
    inp.W[..., 0] = 0.0
    inp.Wsum[:, 0] = 0.0
    head = make_head(inp)
    assert takes_terms(head)
    logphi, logw, _ = oc._params("cp", inp.h, inp.W, inp.Wsum, None)
    want = oc.prefix_marginals_from("cp", logphi, logw, None, inp.targets)
    err = np.abs(head.prefix_marginals(torch.from_numpy(inp.targets).cuda()).cpu().numpy() - want).max()
    print(kept, power, err)
    assert err < LOG * 8 ** 0.5


@pytest.mark.parametrize("B,d,n,r,v", [(257, 512, 8, 11, 33), (513, 544, 4, 20, 320), (300, 1056, 8, 11, 268), (257, 512, 8, 11, 129), (300, 512, 8, 12, 193)])
@pytest.mark.parametrize("where", ["h", "W", "h of infinity in W"])
def test_an_outlier_costs_the_terms_but_not_the_matrix_pipes(where, B, d, n, r, v):
    """Beside a row with an outlier the call goes through three bf16 terms, which hold it; with an infinite weight as well, through
    the fp32 instruction.  Neither gives the bits of a workspace without room for planes, unless that is the same route."""
    inp = mi.make_inputs("cp", B=B, d=d, n=n, r=r, v=v, dtype="f32", seed=v, h_scale=1.0)
    inp.W[..., 0] = 0.0
    inp.Wsum[:, 0] = 0.0
    if where == "W":
        inp.h[:, 0] = 0.0
        inp.W[1, 2, 3, 0] = 2.0 ** 28
    else:
        inp.h[5, 0] = 2.0 ** 28
    logphi, logw, _ = oc._params("cp", inp.h, inp.W, inp.Wsum, None)
    want = oc.prefix_marginals_from("cp", logphi, logw, None, inp.targets)
    if where == "h of infinity in W":
        inp.W[0, 0, 0, 1] = -np.inf
        inp.h[:, 1] = np.abs(inp.h[:, 1]) + 1e-3
        inp.targets[:, 0] = 0                            # a token that one unit rules out
        logphi, logw, _ = oc._params("cp", inp.h, np.where(np.isinf(inp.W), -1e30, inp.W), inp.Wsum, None)
        want = oc.prefix_marginals_from("cp", logphi, logw, None, inp.targets)
    head = make_head(inp)
    assert takes_terms(head)
    tg = torch.from_numpy(inp.targets).cuda()
    got, plain = head.prefix_marginals(tg).cpu().numpy(), without_planes(head, tg).cpu().numpy()
    assert np.abs(got - want).max() < LOG * n ** 0.5
    assert np.abs(plain - want).max() < LOG * n ** 0.5
    assert np.array_equal(got, plain) == (where == "h of infinity in W")


def test_routes_of_a_captured_step():
    """Which terms are due belongs to one pass: a captured scoring call and training step, replayed on plain inputs and on outliers in
    turn, give what eager calls give on the same inputs."""
    B, d, n, r, v = 257, 512, 8, 11, 33
    inp = mi.make_inputs("cp", B=B, d=d, n=n, r=r, v=v, dtype="f32", seed=5, h_scale=1.0)
    head, eager = make_head(inp), make_head(inp)
    assert takes_terms(head)
    eager.h, eager.W = head.h, head.W                         # (the same operands, a workspace of its own)
    tg = torch.from_numpy(inp.targets.astype(np.int32)).cuda()
    coef = torch.from_numpy(bw.loss_coefficients(0.8, np.ones((B, n), bool)).astype(np.float32)).cuda()
    grads = {k: None if t is None else torch.empty_like(t) for k, t in head.loss_backward(tg, coef).items()}
    logq = torch.empty(B, device="cuda")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for _ in range(2):
            head.loglik(tg, out=logq)
            head.loss_backward(tg, coef, out=grads)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        head.loglik(tg, out=logq)
        head.loss_backward(tg, coef, out=grads)
    W5, h5, c0 = head.W[1, 2, 3, 4].clone(), head.h[7, 4].clone(), coef[7, 0].clone()
    seen = []
    for weight, feature, first in ((W5, h5, c0), (W5, 1e6, c0), (W5, h5, c0), (1e6, h5, c0), (W5, 1e25, c0), (W5, h5, c0), (-1e25, h5, c0), (W5, h5, 1e25),
                                   (W5, h5, c0)):
        head.W[1, 2, 3, 4], head.h[7, 4], coef[7, 0] = weight, feature, first
        graph.replay()
        torch.cuda.synchronize()
        want, ref = eager.loglik(tg), eager.loss_backward(tg, coef)
        assert torch.equal(logq.nan_to_num(nan=7.0), want.nan_to_num(nan=7.0))       # (no number where a logit is 1e25)
        for k, t in grads.items():
            if t is not None:
                assert torch.equal(t.nan_to_num(nan=7.0), ref[k].nan_to_num(nan=7.0)), (k, weight, feature, first)
        seen.append(want.clone())
    assert all(torch.equal(seen[0], seen[k]) for k in (2, 5, 8))
