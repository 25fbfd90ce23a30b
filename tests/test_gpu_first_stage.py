"""GPU parity of passes over W whose slabs begin at different stages of K (one tile of positions): one
stage in all, fewer stages than the ring has buffers, fewer and more than there are slabs, on every tile that streams W,
from W's own rows and from either stage-major copy of it (the same bits).

Tolerance: as in test_gpu_tile_positions, sums of d <= 2080 products."""
import numpy as np
import pytest
import torch

import mtpc_inputs as mi
from oracle import mtpc_oracle as oc
from gpu_util import make_head

pytestmark = pytest.mark.gpu

LOG = 4e-5


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [32, 96, 2048, 2080])
@pytest.mark.parametrize("B,r", [(1, 11), (40, 11), (64, 70), (100, 11), (129, 70), (200, 70), (256, 70)])
def test_scores(B, r, d, dtype):
    inp = mi.make_inputs("cp", B=B, d=d, n=4, r=r, v=61, dtype=dtype, seed=B + d, h_scale=1.0)
    logphi, logw, _ = oc._params("cp", inp.h, inp.W, inp.Wsum, None)
    want = oc.prefix_marginals_from("cp", logphi, logw, None, inp.targets)
    head, tg = make_head(inp), torch.from_numpy(inp.targets).cuda()
    got = head.prefix_marginals(tg)
    assert np.abs(got.cpu().numpy() - want).max() < LOG
    if (d * (2 if dtype == "bf16" else 4)) % (128 if B <= 64 else 64) == 0:
        head.pack_W()
        assert torch.equal(head.prefix_marginals(tg), got)


def starts_differ(row_bytes, B):
    """Rows of a multiple of 2 KB or next to one of 8 KB, from 4 KB on; tiles of more than 128 positions: all from there on."""
    return row_bytes >= 4096 and (B > 128 or row_bytes % 2048 == 0 or (row_bytes + 64) % 8192 <= 128)


@pytest.mark.parametrize("dtype,d", [(t, d) for t in ("bf16", "f32") for d in (32, 96, 2048, 2080)] + [("bf16", 2592), ("bf16", 4064)])
@pytest.mark.parametrize("B", [1, 32, 40, 64, 100, 129, 200, 256])
def test_order_of_many_slabs(B, d, dtype):
    """Batches of every tile with more slabs (280) than calls of few tiles have, which take another kernel; sums of d <= 4064 products."""
    r = 70
    inp = mi.make_inputs("cp", B=B, d=d, n=4, r=r, v=61, dtype=dtype, seed=B + d, h_scale=1.0)
    logphi, logw, _ = oc._params("cp", inp.h, inp.W, inp.Wsum, None)
    want = oc.prefix_marginals_from("cp", logphi, logw, None, inp.targets)
    head, tg = make_head(inp), torch.from_numpy(inp.targets).cuda()
    got = head.prefix_marginals(tg)
    assert np.abs(got.cpu().numpy() - want).max() < LOG
    row_bytes = d * (2 if dtype == "bf16" else 4)
    if B >= 32 and not (dtype == "f32" and B > 128):        # (fp32 beyond: products of terms)
        # the order shows beside the table that tokens are drawn from, whose sums begin with K
        table = torch.empty(B, 4, r, 61, dtype=torch.float32, device="cuda")
        head.sample(1, seed=1, logphi=table)
        assert torch.equal(head.table_scores(table, tg, prefix=True), got) == (not starts_differ(row_bytes, B))
    if row_bytes % (128 if B <= 64 else 64) == 0:
        head.pack_W()
        assert torch.equal(head.prefix_marginals(tg), got)
