"""The attention calls whose speed matters, as measurable cases.

A case is one call of the package's public entry points (``ops.attention_forward``
and its variants for inference, ``ops.mra_attention`` with its backward for
training) on inputs made on the GPU. Sizes are the workloads of
``paper_2207_10284_amd.inputs`` and generic ones in between: one short sequence
to sixteen heads of 32768 tokens, both element types, every head width, block
counts that are not multiples of the kernels' groups of 16 rows.
"""
from __future__ import annotations

import math

import torch

from paper_2207_10284_amd import ops

BLOCK = 32


def _case(name, mode, variant, B, H, n, d, dtype, budget, kind, rho=0.95, scales=(), budgets=()):
    c = dict(mode=mode, variant=variant, B=B, H=H, n=n, d=d, dtype=dtype, budget=budget, kind=kind, rho=rho)
    if scales:
        c["scales"] = ",".join(map(str, scales))
        c["budgets"] = ",".join(map(str, budgets))
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one head of one short sequence, float32 inference; latency
        _case("tiny-512", "infer", "mra2", 1, 1, 512, 64, "f32", 4, "iid"),
        # one sequence through a RoBERTa-base attention layer, fine-tuning at batch 1; latency
        _case("seq-512-train", "train", "mra2", 1, 12, 512, 64, "bf16", 8, "ar1", 0.9),
        # RoBERTa-base encoder layer at 512 tokens, a served batch
        _case("base-512", "infer", "mra2", 32, 12, 512, 64, "bf16", 8, "ar1", 0.9),
        # small long-sequence classifier with heavy key columns, float32: inference and training
        _case("small-4096", "infer", "mra2", 16, 2, 4096, 32, "f32", 8, "hub"),
        _case("small-4096-train", "train", "mra2", 16, 2, 4096, 32, "f32", 8, "hub"),
        # float32 training at the widest head, a ragged length (47 blocks)
        _case("wide-1504-train", "train", "mra2", 4, 8, 1504, 128, "f32", 8, "ar1", 0.9),
        # RoBERTa-base encoder layer at 4096 tokens: inference and training
        _case("base-4096", "infer", "mra2", 8, 12, 4096, 64, "bf16", 16, "ar1", 0.95),
        _case("base-4096-train", "train", "mra2", 8, 12, 4096, 64, "bf16", 16, "ar1", 0.95),
        # the head-wide budget with diagonal priors, training, a ragged length (93 blocks)
        _case("global-2976-train", "train", "global", 4, 12, 2976, 64, "bf16", 93 * 11, "ar1", 0.95),
        # four resolutions, float32 inference
        _case("levels-4096", "infer", "levels", 2, 12, 4096, 64, "f32", 16, "ar1", 0.95, (512, 128, 32), (3, 8, 16)),
        # 32k tokens, 16 heads of width 128: inference and training (the largest)
        _case("long-32768", "infer", "mra2", 1, 16, 32768, 128, "bf16", 32, "ar1", 0.98),
        _case("long-32768-train", "train", "mra2", 1, 16, 32768, 128, "bf16", 32, "ar1", 0.98),
    ]


def _tiles(c):
    """Refined 32 x 32 blocks of the whole call."""
    heads, nb = c["B"] * c["H"], c["n"] // BLOCK
    return heads * (c["budget"] + nb if c["variant"] == "global" else nb * c["budget"])


def _cost(c):
    """Work in units of a bfloat16 tile product (float32 matrix cores are 16 times slower)."""
    heads, nb = c["B"] * c["H"], c["n"] // BLOCK
    fine = _tiles(c) * c["d"] * (8 if c["dtype"] == "f32" else 1)
    return (fine + heads * nb * nb * c["d"] / 4) * (3 if c["mode"] == "train" else 1)


def draw(rng):
    top = max(_cost(c) for c in listed())
    while True:
        mode = rng.choice(["infer", "train"])
        dtype = rng.choice(["bf16", "bf16", "f32"])
        variant = rng.choice(["mra2", "mra2", "mra2", "mra2s", "global", "levels"])
        if variant == "levels":
            mode = "infer"                      # the levels path has no backward
        d = rng.choice([32, 64, 64, 128])
        nb = max(4, round(math.exp(rng.uniform(math.log(4), math.log(1024)))))
        heads = max(1, round(math.exp(rng.uniform(math.log(1), math.log(384)))))
        H = rng.choice([h for h in (1, 2, 4, 8, 12, 16) if h <= heads])
        B = max(1, heads // H)
        m = max(1, min(rng.choice([2, 4, 8, 12, 16, 24, 32]), nb // 3))
        kind = rng.choice(["iid", "ar1", "ar1", "hub"])
        rho = rng.choice([0.9, 0.95, 0.98])
        scales, budgets = (), ()
        if variant == "levels":
            nb = max(32, nb // 16 * 16)
            m = min(m, nb // 4)
            if rng.random() < 0.5:
                scales, budgets = (128, 32), (max(m // 2, 2), m)
            else:
                scales, budgets = (512, 128, 32), (max(m // 5 + 1, 2), max(m // 2, 4), m)
            if any(b > nb * BLOCK // s for b, s in zip(budgets, scales)):
                continue
        budget = nb * max(1, m - 1) if variant == "global" else m
        if variant == "global" and budget > nb * (nb - 1):
            continue
        c = _case("", mode, variant, B, H, nb * BLOCK, d, dtype, budget, kind, rho, scales, budgets)
        if _cost(c) <= top and B * H * nb * BLOCK * d <= 96 * 4096 * 128:
            return c


def _torch_dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _ar1(gen, shape, rho, s2):
    """x_t = rho x_{t-1} + e_t along the tokens from a stationary start, by doubling."""
    x = torch.randn(shape, generator=gen, device="cuda") * math.sqrt(s2)
    x[:, :, 0] /= math.sqrt(1.0 - rho * rho)
    step, f = 1, rho
    while step < shape[2] and f > 1e-8:
        y = x.clone()
        y[:, :, step:].add_(x[:, :, :-step], alpha=f)
        x, step, f = y, 2 * step, f * f
    return x


def _inputs(c, seed):
    """q, k, v and the output's gradient: the synthetic kinds of the package's workloads."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(220710284 + seed)
    B, H, n, d = shape = (c["B"], c["H"], c["n"], c["d"])
    if c["kind"] == "ar1":
        s2 = 0.5 if c["rho"] > 0.97 else 1.0
        q, k = _ar1(gen, shape, c["rho"], s2), _ar1(gen, shape, c["rho"], s2)
    else:
        q, k = (torch.randn(shape, generator=gen, device="cuda") for _ in range(2))
    v = torch.randn(shape, generator=gen, device="cuda")
    if c["kind"] == "iid":
        q, k, v = (t * d ** -0.5 for t in (q, k, v))
    if c["kind"] == "hub":
        for b in range(B):
            g = torch.randn(d, generator=gen, device="cuda")
            at = torch.randperm(n, generator=gen, device="cuda")[: round(0.05 * n)]
            k[b, :, at] += 4.0 * g / g.norm()
    g = torch.randn(shape, generator=gen, device="cuda") if c["mode"] == "train" else None
    return tuple(None if t is None else t.to(_torch_dtype(c)) for t in (q, k, v, g))


def _ints(text):
    return tuple(int(s) for s in text.split(","))


def prepare(case, seed):
    q, k, v, g = _inputs(case, seed)
    if case["mode"] == "train":
        q, k, v = (t.requires_grad_(True) for t in (q, k, v))
    state = {"q": q, "k": k, "v": v, "g": g, "mode": case["mode"], "variant": case["variant"],
             "budget": case["budget"]}
    if case["variant"] == "levels":
        state["scales"], state["budgets"] = _ints(case["scales"]), _ints(case["budgets"])
    return state


def run(state):
    q, k, v, m = state["q"], state["k"], state["v"], state["budget"]
    variant = state["variant"]
    if state["mode"] == "train":
        z = ops.mra_attention(q, k, v, m, variant, variant == "global")
        return (z.detach(), *torch.autograd.grad(z, (q, k, v), state["g"]))
    if variant == "mra2":
        return ops.attention_forward(q, k, v, m)
    if variant == "mra2s":
        return ops.sparse_attention_forward(q, k, v, m)
    if variant == "global":
        return ops.attention_forward_global(q, k, v, m, True)
    return ops.attention_forward_levels(q, k, v, state["scales"], state["budgets"])


def work(case):
    heads, nb, n, d = case["B"] * case["H"], case["n"] // BLOCK, case["n"], case["d"]
    elem = 2 if case["dtype"] == "bf16" else 4
    train = case["mode"] == "train"
    # infer: q, k, v in, z out; train: also dz in, dq, dk, dv out
    nbytes = (8 if train else 4) * heads * n * d * elem
    # per refined block two products of 32 x 32 x d forward and five more backward;
    # block logits and the low-resolution term: two and five of nb x nb x d per head
    products = 7 if train else 2
    flops = products * 2 * BLOCK * BLOCK * d * _tiles(case)
    if case["variant"] == "levels":
        flops += sum(4 * heads * (n // s) ** 2 * d for s in _ints(case["scales"]))
    else:
        flops += products * 2 * heads * nb * nb * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # bfloat16: the tile weights, the logit gradients and the results are rounded
    # to bfloat16; measured against float64 0.0019 for z and 0.0070 for dq, whose
    # terms cancel. float32: sums in another order and the exponential of logits
    # of some tens, measured 2.2e-6. Four times that.
    if case["dtype"] == "bf16":
        return {"rel": 3e-2 if case["mode"] == "train" else 1e-2}
    return {"rel": 1e-5}


def _means(x, s):
    return x.view(x.shape[0], -1, s, x.shape[-1]).mean(2)


def _top(S, m):
    """The m largest of each row (equal values: the lower index) as a mask."""
    keep = torch.zeros(S.shape, dtype=torch.bool, device=S.device)
    at = torch.sort(S, dim=-1, descending=True, stable=True).indices[..., :m]
    return keep.scatter_(-1, at, True)


def _wide(t, r, dims=(1, 2)):
    for dim in dims:
        t = t.repeat_interleave(r, dim) if r > 1 else t
    return t


def _level_grid(q, k, case, scale):
    """Per 32-block the coarse logit that stands for it (levels above 32 included) and the refined blocks."""
    scales, budgets = _ints(case["scales"]), _ints(case["budgets"])
    grid, cand, prev = None, None, None
    for s, m in zip(scales, budgets):
        S = _means(q, s) @ _means(k, s).transpose(1, 2) * scale
        if cand is not None:
            cand = _wide(cand, prev // s)
            grid = torch.where(cand, S, _wide(grid, prev // s))
            S = S.masked_fill(~cand, -math.inf)
        else:
            grid = S
        cand, prev = _top(S, m), s
    return grid, cand


def exact(case, seed):
    """The same attention in float64: softmax over the fine logits of the refined
    blocks and the block logits of the others, gradients by autograd with the
    selection held fixed."""
    q, k, v, g = _inputs(case, seed)
    B, H, n, d = q.shape
    nb, scale, variant = n // BLOCK, d ** -0.5, case["variant"]
    train = case["mode"] == "train"
    flat = [None if t is None else t.reshape(B * H, n, d) for t in (q, k, v, g)]
    outs = [torch.empty(B * H, n, d, dtype=torch.float64, device=q.device) for _ in range(4 if train else 1)]
    room = 1 << 25                              # logits held at once
    hs = max(1, min(B * H, room // (n * n)))
    xs = max(1, min(nb, room // (hs * BLOCK * n)))
    for h0 in range(0, B * H, hs):
        Q, K, V = (t[h0:h0 + hs].double().requires_grad_(train) for t in flat[:3])
        with torch.no_grad():
            if variant == "levels":
                grid, keep = _level_grid(Q, K, case, scale)
            else:
                S = _means(Q, BLOCK) @ _means(K, BLOCK).transpose(1, 2) * scale
                if variant == "global":
                    diag = torch.eye(nb, dtype=torch.bool, device=S.device)
                    free = S.masked_fill(diag, -math.inf).flatten(1)
                    keep = _top(free, case["budget"]).view(S.shape) | diag
                else:
                    keep = _top(S, case["budget"])
        for x0 in range(0, nb, xs):
            rows = slice(BLOCK * x0, BLOCK * min(nb, x0 + xs))
            with torch.set_grad_enabled(train):
                logits = Q[:, rows] @ K.transpose(1, 2) * scale
                if variant == "mra2s":
                    low = torch.full_like(keep[:, x0:x0 + xs], -math.inf, dtype=torch.float64)
                elif variant == "levels":
                    low = grid[:, x0:x0 + xs]
                else:
                    low = _means(Q[:, rows], BLOCK) @ _means(K, BLOCK).transpose(1, 2) * scale
                logits = torch.where(_wide(keep[:, x0:x0 + xs], BLOCK), logits, _wide(low, BLOCK))
                z = torch.softmax(logits, -1) @ V
                outs[0][h0:h0 + hs, rows] = z.detach()
                if train:
                    z.backward(flat[3][h0:h0 + hs, rows].double())
        if train:
            for o, t in zip(outs[1:], (Q, K, V)):
                o[h0:h0 + hs] = t.grad
    outs = [o.view(B, H, n, d) for o in outs]
    return tuple(outs) if train else outs[0]
