"""Drafts of a CP of which each is made by workgroups that compute the sum units themselves, against those whose sum units and latents
come from a launch before: a draft's random numbers are its position's and its own, the sums are formed in one order, so that latents and
tokens of draft 0 must be the same, bit for bit, in a call that is small enough and in one that asks for more drafts."""
import pytest
import torch

import mtpc_inputs as mi
from gpu_util import make_head

pytestmark = pytest.mark.gpu


# at most 256 workgroups (n ceil(v / 32) to a draft) and 64 MB of Wsum for them for one draft to a position, more of the one or the other for S
@pytest.mark.parametrize("dtype,B,d,n,r,v,S", [("bf16", 1, 4096, 16, 32, 320, 2), ("bf16", 1, 2080, 16, 63, 268, 4),
                                               ("f32", 1, 1024, 16, 64, 257, 4), ("bf16", 2, 4096, 9, 40, 33, 8),
                                               ("f32", 3, 4096, 3, 100, 65, 10), ("bf16", 1, 96, 64, 128, 9, 64)])
def test_drafts_do_not_depend_on_their_number(dtype, B, d, n, r, v, S):
    head = make_head(mi.make_inputs("cp", B=B, d=d, n=n, r=r, v=v, dtype=dtype, seed=d + r, h_scale=1.0))
    for seed in range(4):
        one, z1, _ = head.sample(1, seed=seed)
        many, zs, _ = head.sample(S, seed=seed)
        assert torch.equal(z1[:, 0], zs[:, 0]) and torch.equal(one[:, 0], many[:, 0])
        assert int(one.min()) >= 0 and int(one.max()) < v


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,n,r,v", [(64, 3, 2, 1), (96, 4, 3, 33), (544, 5, 9, 31), (256, 16, 64, 320), (2080, 8, 65, 32), (32, 2, 128, 64)])
def test_latents_are_those_of_a_call_with_scores(dtype, d, n, r, v):
    head = make_head(mi.make_inputs("cp", B=1, d=d, n=n, r=r, v=v, dtype=dtype, seed=d + r, h_scale=1.0))
    for seed in range(4):
        _, z, _ = head.sample(1, seed=seed)
        _, want, _ = head.sample(1, seed=seed, want_prefix=True)
        assert torch.equal(z, want)
    greedy, z, _ = head.greedy_draft()
    want_t, want, _ = head.greedy_draft(want_prefix=True)
    assert torch.equal(z, want) and torch.equal(greedy, want_t)
