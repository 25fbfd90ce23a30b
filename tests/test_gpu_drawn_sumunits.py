"""The root weights that latents are drawn from, bit for bit: more than 64 units over long bf16 rows in batches of more than 128 positions have
their sums formed along K in one chain, as a pass over a vocabulary of as many tokens forms its logits, so that a seed's latents stay what
they are whatever other form the scores of such a batch take."""
import numpy as np
import pytest
import torch

import mtpc_inputs as mi
from gpu_util import make_head

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,r", [(1056, 65), (1088, 128), (4096, 100), (2080, 97)])
@pytest.mark.parametrize("B", [129, 200, 256])
def test_weights_that_latents_are_drawn_from(B, d, r):
    inp = mi.make_inputs("cp", B=B, d=d, n=1, r=r, v=r, dtype="bf16", seed=d + r, h_scale=1.0)
    one = mi.f32_to_bf16_bits(np.float32([1.0, 200.0]))
    inp.h_bits[:, 0], inp.W_bits[:] = one[0], 0
    inp.W_bits[0, np.arange(r), np.arange(r), 0] = one[1]   # unit k emits token k alone: a draft's score is its weight
    head = make_head(inp)
    S = 16
    drafts, latents, scores = head.sample(S, seed=1, want_prefix=True)
    assert torch.equal(drafts, latents)
    words = mi.make_inputs("ff", B=32, d=d, n=1, r=1, v=r, dtype="bf16", seed=1, h_scale=1.0)
    words.W_bits = inp.Wsum_bits[None, None]
    for b0 in range(0, B, 32):
        nb = min(32, B - b0)
        words.B, words.h, words.h_bits = nb, inp.h[b0:b0 + nb], inp.h_bits[b0:b0 + nb]
        logw = torch.empty(nb, 1, 1, r, dtype=torch.float32, device="cuda")
        make_head(words).sample(1, seed=1, logphi=logw)
        want = logw[:, 0, 0].gather(1, drafts[b0:b0 + nb, :, 0].long())
        assert torch.equal(scores[b0:b0 + nb, :, 0], want)
