"""Drafts drawn from the table that the call leaves (more than 64 positions): the table a seed's tokens are drawn from has the same bits
whatever the number of positions, one tile of them or several, so that a draft does not depend on it."""
import pytest
import torch

import mtpc_inputs as mi
from gpu_util import make_head

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 2048), ("bf16", 2080), ("f32", 1024), ("bf16", 96)])
@pytest.mark.parametrize("B", [65, 100, 129, 200, 256])
def test_a_position_is_drawn_from_the_same_bits(B, dtype, d):
    n, r, v, many = 4, 70, 61, 600
    inp = mi.make_inputs("cp", B=many, d=d, n=n, r=r, v=v, dtype=dtype, seed=d, h_scale=1.0)
    full = make_head(inp)
    want = torch.empty(many, n, r, v, dtype=torch.float32, device="cuda")
    full.sample(1, seed=3, logphi=want)
    inp.h, inp.B = inp.h[:B], B
    inp.h_bits = None if inp.h_bits is None else inp.h_bits[:B]
    head = make_head(inp)
    table = torch.empty(B, n, r, v, dtype=torch.float32, device="cuda")
    drafts, latents, _ = head.sample(1, seed=3, logphi=table)
    assert torch.equal(table, want[:B])
