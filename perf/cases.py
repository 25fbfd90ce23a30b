"""What a user of the head has it do, as cases that can be timed: scoring windows, drafting and verifying
while decoding, marginals, and the training step, each through the public entry points of
``paper_2511_11346_amd.Head``.

A case is a dict of plain values: ``op`` (see ``run``), ``family``, ``dtype`` of h and the weights, the sizes
``B`` (positions), ``d`` (hidden), ``n`` (window), ``r`` (units per layer), ``v`` (vocabulary), whether the
r x r layers are computed from h (``ctx``) and whether the program keeps the stage-major copy of W that
serving with fixed weights makes once (``packed``).
"""
import math

import torch

from paper_2511_11346_amd import Head

OPS = ("prefix", "loglik", "univariate", "greedy", "decode", "draft_score", "train")


def _case(name, op, family, dtype, B, d, n, r, v, ctx=False, packed=False):
    return {"name": name, "op": op, "family": family, "dtype": dtype, "B": B, "d": d, "n": n, "r": r, "v": v,
            "ctx": ctx, "packed": packed}


def listed():
    return [
        # the smallest call: a byte vocabulary scored in fp32 on a small model, where launches and latency count
        _case("prefix_cp_f32_b64", "prefix", "cp", "f32", 64, 256, 4, 8, 256),
        # greedy speculative decoding of one sequence: a draft that needs no scores, and its verification
        _case("greedy_cp_b1", "greedy", "cp", "bf16", 1, 4096, 16, 32, 320, packed=True),
        # one cycle of speculative sampling for one sequence: draft, its prefix scores, verification
        _case("decode_cp_b1", "decode", "cp", "bf16", 1, 4096, 16, 32, 320, packed=True),
        # the same for a server's batch that is not a round number, the head with the longest chain of layers
        _case("decode_hmm_b61", "decode", "hmm", "bf16", 61, 4096, 16, 32, 320),
        # a prompt of a few hundred positions scored: more than a decode batch, less than a training one
        _case("prefix_btree_b200", "prefix", "btree", "bf16", 200, 4096, 16, 32, 320),
        # per-token marginals of a thousand positions
        _case("univariate_hmm_b1000", "univariate", "hmm", "bf16", 1000, 4096, 8, 32, 320),
        # a training-sized batch drafted and scored with fixed weights: targets and drafts in one pass
        _case("draft_score_btree_b4096", "draft_score", "btree", "bf16", 4096, 3072, 16, 64, 320, packed=True),
        # likelihood of a training batch under the fully factorised head (one unit per layer)
        _case("loglik_ff_b8192", "loglik", "ff", "bf16", 8192, 4096, 8, 1, 320),
        # ... and under the HMM whose transitions are computed from the hidden state
        _case("loglik_hmm_ctx_b8192", "loglik", "hmm", "bf16", 8192, 4096, 8, 32, 320, ctx=True),
        # one 2048-byte context of the fp32 byte-level model (a vocabulary that fills no tile)
        _case("loglik_cp_f32_b2048", "loglik", "cp", "f32", 2048, 3072, 8, 32, 268),
        # its training step, loss and all gradients
        _case("train_hmm_f32_b2048", "train", "hmm", "f32", 2048, 3072, 8, 32, 268),
        # the largest: the training step of the tree with 64 units and a window of 16
        _case("train_btree_b4096", "train", "btree", "bf16", 4096, 3072, 16, 64, 320),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_RANGE_B = {"prefix": (1, 8192), "loglik": (1, 8192), "univariate": (16, 4096), "greedy": (1, 8), "decode": (1, 64),
            "draft_score": (65, 8192), "train": (100, 8192)}


def draw(rng):
    """One more case of the same ranges; never more work than the largest listed one (fp32 work counts for
    more, as its matrix instructions are that much slower)."""
    most = max(work(c)["flops"] for c in listed())
    most_bytes = max(work(c)["bytes"] for c in listed())
    while True:
        op = rng.choice(OPS)
        family = rng.choice(("ff", "cp", "hmm", "btree"))
        dtype = "f32" if rng.random() < 0.3 else "bf16"
        d = 32 * max(8, round(_log_uniform(rng, 256, 4096) / 32))
        n = rng.choice((4, 8, 16)) if family == "btree" else rng.randint(3, 16)
        r = 1 if family == "ff" else rng.choice((8, 16, 32, 64, rng.randint(3, 64)))
        v = rng.choice((320, 268, 256, rng.randint(33, 320)))
        lo, hi = _RANGE_B[op]
        c = _case("", op, family, dtype, _log_uniform(rng, lo, hi), d, n, r, v)
        del c["name"]
        esz = 4 if dtype == "f32" else 2
        stage = 128 if c["B"] <= 64 else 64
        if op in ("greedy", "decode", "draft_score"):
            c["packed"] = (d * esz) % stage == 0 and rng.random() < 0.7
        # layers computed from h: of a size that R (r * r * d per layer) still is a weight like W
        c["ctx"] = family in ("hmm", "btree") and r <= 32 and rng.random() < 0.3
        w = work(c)
        if w["flops"] * (16 if dtype == "f32" else 1) <= most and w["bytes"] <= most_bytes:
            return c


def _n_layers(case):
    return {"hmm": case["n"] - 1, "btree": case["n"] - 2}.get(case["family"], 0)


def _inputs(case, seed):
    """Device tensors of one head and one batch.  h is what a normalised hidden state looks like (unit
    variance), W gives logits of standard deviation 2 (a byte model's predictions are peaked), the layers are those
    of a head that was initialised at the identity and has moved away from it (about 0.6 on the diagonal)."""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    B, d, n, r, v = (case[k] for k in "Bdnrv")
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16

    def gauss(*shape, std=1.0, dtype=dt):
        return torch.randn(*shape, generator=gen, device=dev, dtype=dtype).mul_(std)

    h = gauss(B, d)
    W = gauss(n, r, v, d, std=2.0 / math.sqrt(d))
    Wsum = None if case["family"] == "ff" else gauss(r, d, std=1.0 / math.sqrt(d))
    L = _n_layers(case)
    layers = R = None
    if L > 0:
        eye = (math.log(r) + 1.0) * torch.eye(r, device=dev, dtype=torch.float32)
        if case["ctx"]:
            R = gauss(L, r, r, d, std=1.0 / math.sqrt(d))
            layers = eye.expand(L, r, r).contiguous()
        else:
            layers = eye + gauss(L, r, r, dtype=torch.float32)
    x = {"h": h, "W": W, "Wsum": Wsum, "layers": layers, "R": R,
         "targets": torch.randint(0, min(v, 256), (B, n), generator=gen, device=dev, dtype=torch.int32)}
    if case["op"] in ("greedy", "decode"):
        x["p"] = torch.softmax(gauss(B, n + 1, v, std=2.0, dtype=torch.float32), dim=-1).contiguous()
    if case["op"] == "train":
        # discounted loss over the positions whose window is whole
        valid = (torch.rand(B, n, generator=gen, device=dev) < 0.9).float()
        x["coef"] = (0.8 ** torch.arange(n, device=dev, dtype=torch.float32) * valid / valid.sum()).contiguous()
    return x


def prepare(case, seed):
    """The head and what its program keeps beside it: buffers for the table, for the gradients."""
    x = _inputs(case, seed)
    h, W, Wsum, layers, R = (x[k] for k in ("h", "W", "Wsum", "layers", "R"))
    B, d, n, r, v = (case[k] for k in "Bdnrv")
    head = Head(case["family"], h, W, Wsum, layers, R)
    if case["packed"]:
        head.pack_W()
    f32 = {"dtype": torch.float32, "device": h.device}
    state = {"case": case, "head": head, "seed": seed & 0x7fffffff}
    state.update({k: x[k] for k in ("targets", "p", "coef") if k in x})
    if case["op"] == "decode":
        state["table"] = torch.empty(B, n, r, v, **f32)
    if case["op"] == "train":
        state["grads"] = {"loss": torch.empty(B, **f32), "dh": torch.empty(B, d, **f32), "dW": torch.empty(n, r, v, d, **f32),
                          "dWsum": None if Wsum is None else torch.empty(r, d, **f32),
                          "dlayers": None if layers is None else torch.empty_like(layers),
                          "dR": None if R is None else torch.empty(R.shape, **f32)}
    return state


def run(state):
    """One pass: the call, or the calls of one cycle, as a user's program makes them."""
    head, op = state["head"], state["case"]["op"]
    if op == "loglik":
        return head.loglik(state["targets"])
    if op == "prefix":
        return head.prefix_marginals(state["targets"])
    if op == "univariate":
        return head.univariate_marginals()
    if op == "greedy":
        drafts, _, _ = head.greedy_draft(want_latents=False)
        accepted, token = head.verify(drafts, state["p"], mode="greedy")
        return drafts, accepted, token
    if op == "decode":
        drafts, _, scores = head.sample(1, seed=state["seed"], want_latents=False, want_prefix=True, logphi=state["table"])
        accepted, token = head.verify(drafts[:, 0], state["p"], prefix_logq=scores[:, 0], logphi=state["table"],
                                      seed=state["seed"], offset=1)
        return drafts, scores, state["table"], accepted, token
    if op == "draft_score":
        drafts, latents, _ = head.sample(1, seed=state["seed"])
        return drafts, latents, head.window_scores(state["targets"][:, None], drafts, prefix=True)
    out = head.loss_backward(state["targets"], state["coef"], out=state["grads"])
    return {k: t for k, t in out.items() if t is not None}


def work(case):
    B, d, n, r, v, op = (case[k] for k in ("B", "d", "n", "r", "v", "op"))
    esz = 4 if case["dtype"] == "f32" else 2
    L = _n_layers(case)
    W, h = n * r * v * d * esz, B * d * esz
    small = 0 if case["family"] == "ff" else r * d * esz
    small += L * r * r * (4 + (d * esz if case["ctx"] else 0))
    layers = 2 * B * L * r * r * d if case["ctx"] else 0
    full = 2 * B * n * r * v * d + layers
    ids = B * n * 4
    if op == "greedy":
        # only the slabs of W that the drafts' tokens are drawn from
        return {"bytes": min(B, r) * n * v * d * esz + h + small + B * (n + 1) * v * 4 + ids, "flops": 2 * B * n * v * d + layers}
    if op == "decode":
        return {"bytes": W + h + small + B * n * r * v * 4 + B * (n + 1) * v * 4 + 2 * ids, "flops": full}
    if op == "draft_score":
        return {"bytes": W + h + small + 4 * ids, "flops": full + 2 * B * n * v * d}
    if op == "univariate":
        return {"bytes": W + h + small + B * n * v * 4, "flops": full}
    if op == "train":
        # the gradients are fp32: the weights' and h's once more, at four bytes
        return {"bytes": W + h + small + ids * 2 + (n * r * v + B + r) * d * 4 + L * r * r * 4 * (d + 1 if case["ctx"] else 1),
                "flops": 3 * full}
    return {"bytes": W + h + small + 2 * ids, "flops": full}


def tolerance(case):
    if case["op"] in ("greedy", "decode", "draft_score"):
        # tokens are whole values: a uniform (or two most likely tokens) within fp32 rounding of a boundary may go
        # either way, and then the scores of that draft are another draft's
        return {"rel": 2e-3, "max": 0.5, "differ": 1e-4}
    # measured against the same path in 64 bits, times about four: gradients 4e-6 of their norm with fp32 inputs and
    # 1.7e-3 with bf16 ones (the logit gradient is rounded to bf16 once), logs of probabilities 1.3e-7
    if case["op"] == "train":
        return {"rel": 7e-3, "max": 0.4} if case["dtype"] == "bf16" else {"rel": 2e-5}
    return {"rel": 1e-6}


# ---- the same values in 64 bits, in plain torch -------------------------------------------------------------

def _lse_step(A, x):
    """log sum_j exp(A[.., k, j]) exp(x[b, j]); A [k, j] shared or [b, k, j] of each position."""
    m = x.amax(dim=-1, keepdim=True)
    w = torch.exp(x - m)
    y = w @ torch.exp(A).T if A.dim() == 2 else (torch.exp(A) * w[:, None, :]).sum(dim=-1)
    return m + torch.log(y)


def _joint(family, e, logw, logA):
    """log of the circuit's value from the log evidence e [B, n, r]; layer l of logA is logA[l] or logA[:, l]."""
    n = e.shape[1]
    layer = (lambda l: logA[l]) if logA is None or logA.dim() == 3 else (lambda l: logA[:, l])
    if family == "ff":
        return e[:, :, 0].sum(dim=1)
    if family == "cp":
        return torch.logsumexp(logw + e.sum(dim=1), dim=-1)
    if family == "hmm":
        alpha = logw + e[:, 0]
        for i in range(1, n):
            alpha = e[:, i] + _lse_step(layer(i - 1).transpose(-1, -2), alpha)
        return torch.logsumexp(alpha, dim=-1)
    node = [None] * (n - 1) + [e[:, i] for i in range(n)]
    for m in range(n - 2, 0, -1):
        node[m] = _lse_step(layer(m - 1), node[2 * m + 1] + node[2 * m + 2])
    return torch.logsumexp(logw + node[1] + node[2], dim=-1)


def _prefix(family, e, logw, logA):
    n = e.shape[1]
    past = torch.tril(torch.ones(n, n, dtype=e.dtype, device=e.device))
    return torch.stack([_joint(family, e * past[i][None, :, None], logw, logA) for i in range(n)], dim=1)


def _leaf_marginals(family, logw, logA, n, B):
    """log of the marginal of the latent that selects the input units of each token: [B, n, r]."""
    if family == "ff":
        return torch.zeros(B, n, 1, dtype=torch.float64, device="cuda:0")
    if family == "cp":
        return logw[:, None, :].expand(B, n, logw.shape[-1])
    layer = (lambda l: logA[l].transpose(-1, -2)) if logA is None or logA.dim() == 3 else (lambda l: logA[:, l].transpose(-1, -2))
    if family == "hmm":
        z = [logw]
        for i in range(1, n):
            z.append(_lse_step(layer(i - 1), z[-1]))
        return torch.stack(z, dim=1)
    z = [logw]
    for m in range(1, n - 1):
        z.append(_lse_step(layer(m - 1), z[(m - 1) // 2]))
    return torch.stack([z[(n - 2 + i) // 2] for i in range(n)], dim=1)


def exact(case, seed):
    """The values of run() that do not depend on a draw."""
    op, family = case["op"], case["family"]
    if op in ("greedy", "draft_score"):
        return None         # whole values, and the scores of what was drawn
    x = _inputs(case, seed)
    B, d, n, r, v = (case[k] for k in "Bdnrv")
    up = lambda t: None if t is None else t.double()
    h, W, tg = x["h"].double(), x["W"], x["targets"].long()
    s = None if x["Wsum"] is None else (h @ up(x["Wsum"]).T).requires_grad_(op == "train")
    lay = up(x["layers"])
    if x["R"] is not None:
        L = x["R"].shape[0]
        lay = lay + torch.stack([h @ up(x["R"][l]).reshape(r * r, d).T for l in range(L)], dim=1).view(B, L, r, r)
    if lay is not None:
        lay = lay.detach().requires_grad_(op == "train")
    logw = None if s is None else torch.log_softmax(s, dim=-1)
    logA = None if lay is None else torch.log_softmax(lay, dim=-1)

    def logphi(i, j):
        return torch.log_softmax(h @ W[i, j].double().T, dim=-1)

    if op == "decode":
        return None, None, torch.stack([torch.stack([logphi(i, j) for j in range(r)], dim=1) for i in range(n)], dim=1), None, None
    if op == "univariate":
        m = _leaf_marginals(family, logw, logA, n, B)
        out = torch.full((B, n, v), -math.inf, dtype=torch.float64, device=h.device)
        for i in range(n):
            for j in range(r):
                out[:, i] = torch.logaddexp(out[:, i], m[:, i, j, None] + logphi(i, j))
        return out
    e = torch.stack([torch.stack([logphi(i, j).gather(1, tg[:, i, None])[:, 0] for j in range(r)], dim=1) for i in range(n)], dim=1)
    if op == "loglik":
        return _joint(family, e, logw, logA)
    if op == "prefix":
        return _prefix(family, e, logw, logA)
    e.requires_grad_(True)
    P = _prefix(family, e, logw, logA)
    loss = (x["coef"].double() * (torch.nn.functional.pad(P[:, :-1], (1, 0)) - P)).sum(dim=1)
    loss.sum().backward()
    out = {"loss": loss.detach(), "dh": torch.zeros(B, d, dtype=torch.float64, device=h.device),
           "dW": torch.empty(n, r, v, d, dtype=torch.float64, device=h.device)}
    for i in range(n):
        for j in range(r):
            g = -torch.exp(logphi(i, j))
            g.scatter_add_(1, tg[:, i, None], torch.ones_like(g[:, :1]))
            g *= e.grad[:, i, j, None]
            out["dW"][i, j] = g.T @ h
            out["dh"] += g @ W[i, j].double()
    if s is not None:
        out["dWsum"] = s.grad.T @ h
        out["dh"] += s.grad @ up(x["Wsum"])
    if x["R"] is not None:
        g = lay.grad.view(B, -1, r * r)
        out["dR"] = torch.stack([(g[:, l].T @ h).view(r, r, d) for l in range(L)])
        out["dlayers"] = lay.grad.sum(dim=0)
        for l in range(L):
            out["dh"] += g[:, l] @ up(x["R"][l]).reshape(r * r, d)
    elif lay is not None:
        out["dlayers"] = lay.grad
    return out
