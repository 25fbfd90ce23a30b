"""GPU parity of calls so small that all tiles of 16 or 32 positions run at once, whose sum units and layers are computed by the launch
that passes over W where they run at once with the others: up to n r ceil(B / 16) = 256 tiles in fp32, n r ceil(B / 32) = 256 beyond that,
and (r > 1) for B <= 16 (n r + 1) ceil(B / 16), for others (n r + 1) ceil(B / 32) = 256 in bf16.  Batches at the edges of a tile and of the rule, vocabularies and units at the edges of the waves' rows (more
units than tokens among them), rows of h and W of one stage, of whole 128-byte stages and of none.

Tolerances: those of the other parity tests."""
import numpy as np
import pytest
import torch

import mtpc_inputs as mi
from oracle import mtpc_oracle as oc
from gpu_util import make_head, oracle_params, tol_check

pytestmark = pytest.mark.gpu

# (B, d, n, r, v)
SIZES = [(1, 32, 3, 7, 5), (16, 64, 4, 8, 33), (17, 96, 4, 8, 128), (32, 160, 3, 21, 129), (33, 256, 4, 7, 256), (64, 256, 4, 8, 257),
         (1, 1056, 5, 51, 320), (16, 128, 2, 127, 60), (31, 64, 2, 128, 5), (63, 128, 3, 17, 268), (100, 192, 4, 8, 100),
         (160, 96, 8, 3, 320), (250, 64, 2, 7, 63), (300, 32, 8, 3, 17), (500, 128, 4, 2, 200), (257, 512, 7, 2, 320),
         (64, 64, 8, 8, 40), (13, 128, 2, 128, 300), (256, 64, 4, 8, 90), (500, 64, 4, 4, 33)]       # (no room for the sum units)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,d,n,r,v", SIZES)
def test_scores_and_marginals(B, d, n, r, v, dtype):
    for family in ("ff", "cp", "hmm", "btree"):
        if family == "btree" and n & (n - 1):
            continue
        inp = mi.make_inputs(family, B=B, d=d, n=n, r=1 if family == "ff" else r, v=v, dtype=dtype, seed=B + d, h_scale=1.0)
        logphi, logw, lay = oracle_params(inp)
        head = make_head(inp)
        x = inp.targets.astype(np.int32).copy()
        x[0, 0], x[-1, -1] = -1, v                          # one variable summed out, one id that is none
        y = np.ascontiguousarray(x[:, ::-1])
        want = {k: oc.prefix_marginals_from(family, logphi, logw, lay, t) for k, t in (("x", x), ("y", y))}
        tx, ty = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
        tol_check(head.prefix_marginals(tx).cpu().numpy(), want["x"], dtype, family)
        # three windows per position, from two places
        three = head.window_scores(torch.stack([tx, ty], dim=1).contiguous(), tx[:, None].contiguous(), prefix=True).cpu().numpy()
        for k, t in enumerate("xyx"):
            tol_check(three[:, k], want[t], dtype, f"{family}, window {k}")
        lay_in = inp.layers
        tol_check(head.univariate_marginals().cpu().numpy(), oc.univariate_marginals(family, inp.h, inp.W, inp.Wsum, lay_in), dtype,
                  f"{family}, marginals")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("family", ["hmm", "btree"])
def test_layers_of_every_position(family, dtype):
    inp = mi.make_inputs(family, B=40, d=64, n=4, r=6, v=50, dtype=dtype, seed=9, h_scale=1.0)
    lay = np.random.default_rng(1).standard_normal((40,) + inp.layers.shape)
    logphi, logw, ll = oc._params(family, inp.h, inp.W, inp.Wsum, lay)
    got = make_head(inp, layers=lay).prefix_marginals(torch.from_numpy(inp.targets).cuda()).cpu().numpy()
    tol_check(got, oc.prefix_marginals_from(family, logphi, logw, ll, inp.targets), dtype, family)


@pytest.mark.parametrize("dtype,d", [("bf16", 2048), ("f32", 1024)])
@pytest.mark.parametrize("B", [1, 16])
def test_a_vocabulary_that_is_streamed(B, d, dtype):
    """More than 128 MB of W and one tile of positions: read as a stream, slabs from different stages of K on."""
    inp = mi.make_inputs("cp", B=B, d=d, n=4, r=36, v=300, dtype=dtype, seed=B, h_scale=1.0)
    logphi, logw, _ = oc._params("cp", inp.h, inp.W, inp.Wsum, None)
    got = make_head(inp).prefix_marginals(torch.from_numpy(inp.targets).cuda()).cpu().numpy()
    tol_check(got, oc.prefix_marginals_from("cp", logphi, logw, None, inp.targets), dtype)


@pytest.mark.parametrize("dtype,d,B", [("bf16", 2048, 17), ("bf16", 2048, 32), ("f32", 1024, 17), ("f32", 1024, 32)] +
                         [("bf16", 2080, B) for B in (1, 16, 17, 32)])       # (rows of 64-byte stages)
def test_a_streamed_vocabulary_in_wider_tiles_and_shorter_stages(B, d, dtype):
    inp = mi.make_inputs("cp", B=B, d=d, n=4, r=36, v=300, dtype=dtype, seed=B, h_scale=1.0)
    logphi, logw, _ = oc._params("cp", inp.h, inp.W, inp.Wsum, None)
    got = make_head(inp).prefix_marginals(torch.from_numpy(inp.targets).cuda()).cpu().numpy()
    tol_check(got, oc.prefix_marginals_from("cp", logphi, logw, None, inp.targets), dtype)
