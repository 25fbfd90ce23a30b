"""Host-side checks of the scratch a call is asked for and accepted with; no GPU: every call here either only
asks for a size or is refused before its first launch."""
import ctypes as C

import pytest
import torch

from paper_2511_11346_amd import binding

HEADS = [("btree", 4096, 3072, 16, 64, 320), ("hmm", 8192, 4096, 8, 32, 320), ("hmm", 1000, 4096, 8, 32, 320), ("cp", 300, 1056, 8, 32, 268)]


def bare_head(family, B, d, n, r, v, dtype):
    """A Head that knows its sizes and has no tensors but an empty h of its dtype."""
    head = binding.Head.__new__(binding.Head)
    head.family, head.B, head.d, head.n, head.r, head.v = family, B, d, n, r, v
    head.h = torch.empty(0, d, dtype=torch.bfloat16 if dtype == binding.BF16 else torch.float32)
    head._sl = binding.mtpc_sumlayers(0x6000, r * r, 0) if family in ("hmm", "btree") else None
    return head


def c_head(B, d, n, r, v, dtype, **kw):
    hd = binding.mtpc_head()
    hd.B, hd.d, hd.n, hd.r, hd.v, hd.dtype = B, d, n, r, v, dtype
    hd.h, hd.ld_h, hd.W, hd.Wsum = 0x1000, d, 0x2000, 0x3000
    for k, x in kw.items():
        setattr(hd, k, x)
    return hd


@pytest.mark.parametrize("dtype", [binding.BF16, binding.F32])
@pytest.mark.parametrize("family,B,d,n,r,v", HEADS)
def test_head_asks_for_the_scratch_of_its_own_dtype(family, B, d, n, r, v, dtype):
    head = bare_head(family, B, d, n, r, v, dtype)
    hd = c_head(B, d, n, r, v, dtype)
    for op in (binding.OP_LOGLIK, binding.OP_MARGINALS, binding.OP_SAMPLE, binding.OP_VERIFY, binding.OP_BACKWARD, binding.OP_WINDOWS):
        for mode in (0, 1):
            want = binding.lib().mtpc_workspace_bytes(binding.FAMILY[family], op, C.byref(hd), head._layers_ref(), 1, mode)
            assert head.workspace_bytes(op, mode=mode) == want > 0


@pytest.mark.parametrize("B,d,n,r,v", [(300, 512, 8, 32, 40), (2048, 3072, 8, 32, 268)])
def test_sampling_has_no_planes(B, d, n, r, v):
    """fp32 draws never go through the planes of the terms (6 bytes per element of W): the static scratch holds none, and
    sampling from it gives the bits of sampling from a workspace."""
    hd = c_head(B, d, n, r, v, binding.F32)
    planes = 6 * n * r * v * d
    size = lambda op: binding.lib().mtpc_workspace_bytes(binding.CP, op, C.byref(hd), None, 1, 0)
    assert size(binding.OP_SAMPLE) < planes < size(binding.OP_LOGLIK)


def test_training_scratch_holds_one_layout_of_the_gradient():
    """A large bf16 step reads W and the logit gradient along their rows: beside the probabilities and that one layout its scratch
    has no room for the other layout or a transpose of W, each of the size of dL [B][n r v]."""
    B, d, n, r, v = 4096, 3072, 16, 64, 320
    M, layers = n * r * v, binding.mtpc_sumlayers(0x6000, r * r, 0)
    hd = c_head(B, d, n, r, v, binding.BF16)
    size = binding.lib().mtpc_workspace_bytes(binding.BTREE, binding.OP_BACKWARD, C.byref(hd), C.byref(layers), 1, 0)
    assert M * B * 6 < size < M * B * 6 + min(M * B, M * d) * 2
