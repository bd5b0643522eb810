"""The work this library is used for, as cases that can be prepared, run once and checked.

A case is one call sequence of a user's program through the public Python entry points:

* ``step``: a training step of the vocabulary projection, ``vp_ce_forward`` then
  ``vp_ce_backward`` on buffers the program keeps (workspace, loss, lse, dH, dW), optionally
  adding into a dW that arrives with other ranks' contributions (``accumulate``);
* ``forward``: the loss of a batch without gradients (``forward``, which allocates its outputs);
* ``noalloc``: the same for a serving loop that may not allocate (``vp_ce_forward_noalloc``);
* ``fold``: the move-activations form of the ring, a fresh state that meets every shard in ring
  order (``new_state``, ``fold_shard`` per shard, ``fold_finalize``).

Sizes are those of ``workloads.py`` where a workload has them; inputs follow its recipe (H
standard normal times a scale, W standard normal over sqrt(d), uniform or Zipf targets, a share
of ignored tokens), drawn on the GPU from the seed.
"""
from __future__ import annotations

import math

import torch

import paper_2609_14306_amd as vp

IGNORE = -100


def _case(name, mode, dtype, T, d, V, P, *, zipf=0.0, ignored=0.0, h_scale=1.0, ragged=False,
          order="natural", accumulate=False):
    return {"name": name, "mode": mode, "dtype": dtype, "T": T, "d": d, "V": V, "P": P, "zipf": zipf,
            "ignored": ignored, "h_scale": h_scale, "ragged": ragged, "order": order,
            "accumulate": accumulate}


def listed():
    return [
        # The smallest call: the tiny float32 workload (unit tests, toy models), where launches
        # and latency are all there is.
        _case("step_tiny_f32", "step", "f32", 256, 256, 2048, 8, ignored=0.05),
        # Scoring one short continuation in a serving loop (d, V and shards of the stress
        # workload): the weights are read for a few tokens.
        _case("score_short_bf16", "noalloc", "bf16", 40, 4096, 151936, 16),
        # Perplexity of one 2k-token document on the wide workload's projection.
        _case("eval_2k_bf16", "forward", "bf16", 2048, 7168, 129280, 8, ignored=0.01),
        # A micro-batch of one short sequence: a training step with few tokens per pass.
        _case("step_512_bf16", "step", "bf16", 512, 2880, 201088, 8, ignored=0.02),
        # One 4096-token sequence (the workload of that name).
        _case("step_4k_bf16", "step", "bf16", 4096, 2880, 201088, 8, ignored=0.02),
        # The long-context workload, the configuration of the benchmark.
        _case("step_longctx_bf16", "step", "bf16", 32768, 2880, 201088, 8, zipf=1.1, order="ring0"),
        # The wide workload: a large hidden width.
        _case("step_wide_bf16", "step", "bf16", 16384, 7168, 129280, 8, ignored=0.01),
        # The stress workload, the largest: 64k tokens, large logits, 16 shards, skewed targets.
        _case("step_stress_bf16", "step", "bf16", 65536, 4096, 151936, 16, zipf=1.3, ignored=0.1,
              h_scale=6.18, order="ring0_reversed"),
        # The paper's float32 projection (hidden 7168, V = 200000 over 8 shards) with 2048 of its
        # tokens.
        _case("step_paper_f32", "step", "f32", 2048, 7168, 200000, 8, order="ring0"),
        # Move-activations ring: 4096 visiting tokens meet eight resident shards one by one.
        _case("fold_4k_bf16", "fold", "bf16", 4096, 2880, 201088, 8, ignored=0.02, order="ring0"),
        # Nothing on a tile boundary: packed tokens without padding, a hidden width that is no
        # multiple of 64, a small tokenizer in uneven shards, and a dW that travels with its shard.
        _case("step_ragged_bf16", "step", "bf16", 1333, 1000, 32003, 5, ignored=0.1, ragged=True,
              order="ring0", accumulate=True),
    ]


# Matrix operations of the largest listed case of each type, the most that a drawn one may cost.
_MOST = {"bf16": 8 * 65536 * 4096 * 151936, "f32": 8 * 2048 * 7168 * 200000}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    mode = rng.choice(["step", "step", "step", "forward", "noalloc", "fold"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    T = _log_int(rng, 40 if mode in ("step", "fold") else 1, 65536)
    V = _log_int(rng, 2048, 201088)
    d = _log_int(rng, 256, 7168)
    d = d // 8 * 8 if rng.random() < 0.25 else max(256, d // 64 * 64)
    per_token = (8 if mode == "step" else 2) * V * d
    T = min(T, max(1, _MOST[dtype] // per_token))
    P = rng.choice([1, 2, 4, 5, 8, 16])
    zipf = rng.choice([0.0, 1.1, 1.3])
    return {"mode": mode, "dtype": dtype, "T": T, "d": d, "V": V, "P": P, "zipf": zipf,
            "ignored": rng.choice([0.0, 0.02, 0.1]), "h_scale": rng.choice([1.0, 1.0, 6.18]),
            "ragged": rng.random() < 0.3, "order": rng.choice(["natural", "ring0", "ring0_reversed"]),
            "accumulate": mode == "step" and rng.random() < 0.3}


# ---------------------------------------------------------------------------------------------
def _rows(case):
    """Shard sizes: ceil(V / P) each and the last one shorter, or uneven ones."""
    V, P = case["V"], case["P"]
    if not case["ragged"]:
        per = -(-V // P)
        return [max(0, min(per, V - p * per)) for p in range(P)]
    weight = [3 + (5 * p) % 7 for p in range(P)]
    cut = [V * sum(weight[:p]) // sum(weight) for p in range(P + 1)]
    return [cut[p + 1] - cut[p] for p in range(P)]


def _order(case):
    P = case["P"]
    if case["order"] == "natural":
        return list(range(P))
    ring = [(-i) % P for i in range(P)]
    return ring if case["order"] == "ring0" else ring[::-1]


def _inputs(case, seed):
    """H, shards, targets, upstream gradient and the dW that a ring brings along (or None)."""
    T, d, V = case["T"], case["d"], case["V"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(n, scale, to):
        return (torch.randn(n, d, generator=gen, device="cuda") * scale).to(to)

    H = normal(T, case["h_scale"], dt)
    rows = _rows(case)
    Ws = [normal(r, 1.0 / math.sqrt(d), dt) for r in rows]
    if case["zipf"]:
        cdf = torch.cumsum(torch.arange(1, V + 1, dtype=torch.float64, device="cuda") ** -case["zipf"], 0)
        u = torch.rand(T, generator=gen, dtype=torch.float64, device="cuda") * cdf[-1]
        targets = torch.searchsorted(cdf, u, right=True).clamp_(max=V - 1)
    else:
        targets = torch.randint(0, V, (T,), generator=gen, device="cuda")
    n_ign = int(round(case["ignored"] * T))
    if n_ign:
        targets[torch.randperm(T, generator=gen, device="cuda")[:n_ign]] = IGNORE
    # the gradient of a mean over the tokens that count, with per-token weights around 1
    g = (0.5 + torch.rand(T, generator=gen, device="cuda")) / max(1, T - n_ign)
    dWs = None
    if case["accumulate"]:  # about the size of one rank's own contribution to a typical row
        scale = case["h_scale"] / math.sqrt(max(1, T) * V)
        dWs = [normal(r, scale, torch.float32) for r in rows]
    return H, Ws, targets.to(torch.int64), g, dWs


def prepare(case, seed):
    H, Ws, targets, g, dWs = _inputs(case, seed)
    order = _order(case)
    T, d, mode = case["T"], case["d"], case["mode"]
    s = {"mode": mode, "H": H, "Ws": Ws, "targets": targets, "order": order}
    if mode == "fold":
        s["rows"] = _rows(case)
        s["offset"] = [sum(s["rows"][:p]) for p in range(case["P"])]
        one = vp.problem_for(H, Ws, IGNORE)  # the size depends on T, d and the type only
        s["ws"] = torch.empty(vp.vp_ce_workspace_size(one)[0], dtype=torch.uint8, device="cuda")
    if mode in ("step", "noalloc"):
        flags = vp.VP_ACCUMULATE_DW if case["accumulate"] else 0
        s["prob"] = vp.problem_for(H, Ws, IGNORE, order, flags)
        s["loss"] = torch.empty(T, dtype=torch.float32, device="cuda")
        s["lse"] = torch.empty(T, dtype=torch.float32, device="cuda")
    if mode == "step":
        s["ws"] = torch.empty(max(vp.vp_ce_workspace_size(s["prob"])), dtype=torch.uint8, device="cuda")
        s["g"] = g
        s["dH"] = torch.empty(T, d, dtype=torch.float32, device="cuda")
        s["dWs"] = dWs or [torch.empty(w.shape[0], d, dtype=torch.float32, device="cuda") for w in Ws]
    return s


def run(s):
    mode = s["mode"]
    if mode == "forward":
        loss, lse = vp.forward(s["H"], s["Ws"], s["targets"], IGNORE, s["order"])
        return {"loss": loss, "lse": lse}
    if mode == "noalloc":
        vp.vp_ce_forward_noalloc(s["prob"], s["H"], s["Ws"], s["targets"], s["loss"], s["lse"])
        return {"loss": s["loss"], "lse": s["lse"]}
    if mode == "fold":
        T = s["H"].shape[0]
        state = vp.new_state(T, s["H"].device)
        for q in s["order"]:
            vp.fold_shard(s["H"], s["Ws"][q], s["offset"][q], s["targets"], state, s["ws"])
        loss, lse = vp.fold_finalize(s["targets"], state, s["rows"], IGNORE, s["ws"])
        return {"loss": loss, "lse": lse, "m": state[:T], "s": state[T:2 * T], "y": state[2 * T:]}
    vp.vp_ce_forward(s["prob"], s["H"], s["Ws"], s["targets"], s["loss"], s["lse"], s["ws"])
    vp.vp_ce_backward(s["prob"], s["H"], s["Ws"], s["targets"], s["lse"], s["g"], s["dH"], s["dWs"],
                      s["ws"])
    return {"loss": s["loss"], "lse": s["lse"], "dH": s["dH"], "dW": s["dWs"]}


def work(case):
    """One read of H, W, targets (and g), one write of every output; the backward starts from lse
    alone, so its products are the recomputed logits, dH and dW."""
    T, d, V = case["T"], case["d"], case["V"]
    e = 2 if case["dtype"] == "bf16" else 4
    nbytes = (T + V) * d * e + 8 * T + 8 * T
    if case["mode"] == "fold":
        nbytes += 12 * T
    if case["mode"] != "step":
        return {"bytes": nbytes, "flops": 2 * T * V * d}
    nbytes += 4 * T + 4 * d * (T + V * (2 if case["accumulate"] else 1))
    return {"bytes": nbytes, "flops": 8 * T * V * d}


def tolerance(case):
    """Losses and fold states are float32 sums, and float32 gradients too (2.9e-6 off the float64
    result at d = 7168, V = 200000); a fold's s carries the rounding of m, an exponent (7e-6 for
    logits near 40); bfloat16 gradients carry the rounding of the residual to bfloat16 (1.7e-3)."""
    if case["mode"] == "step" and case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 0.3}
    if case["mode"] == "fold":
        return {"rel": 3e-5, "max": 1e-3}
    return {"rel": 1.2e-5, "max": 1e-3}


def exact(case, seed):
    """The definitions in float64 on the GPU, a block of vocabulary rows at a time."""
    H, Ws, targets, g, dWs = _inputs(case, seed)
    T, d = case["T"], case["d"]
    H64 = H.double()
    rows = _rows(case)
    off = [sum(rows[:p]) for p in range(case["P"])]
    block = max(256, min(8192, (1 << 29) // max(T, 1)))
    m = torch.full((T,), -math.inf, dtype=torch.float64, device="cuda")
    z = torch.zeros(T, dtype=torch.float64, device="cuda")
    y = torch.zeros(T, dtype=torch.float64, device="cuda")

    def blocks():
        for p, W in enumerate(Ws):
            for r in range(0, W.shape[0], block):
                yield p, r, off[p] + r, W[r:r + block].double()

    def owned(lo, n):
        return ((targets >= lo) & (targets < lo + n)).nonzero().flatten()

    for p, r, lo, W in blocks():
        L = H64 @ W.t()
        t = owned(lo, W.shape[0])
        y[t] = L[t, targets[t] - lo]
        top = torch.maximum(m, L.amax(1))
        z = z * torch.exp(m - top) + torch.exp_(L.sub_(top[:, None])).sum(1)
        m = top
    lse = m + torch.log(z)
    live = targets != IGNORE
    loss = torch.where(live, lse - y, torch.zeros_like(lse))
    if case["mode"] == "fold":
        return {"loss": loss, "lse": lse, "m": m, "s": z, "y": y}
    if case["mode"] != "step":
        return {"loss": loss, "lse": lse}
    g64 = torch.where(live, g.double(), torch.zeros_like(lse))
    dH = torch.zeros(T, d, dtype=torch.float64, device="cuda")
    dW = [torch.zeros(r, d, dtype=torch.float64, device="cuda") if dWs is None else dWs[p].double()
          for p, r in enumerate(rows)]
    for p, r, lo, W in blocks():
        G = torch.exp_((H64 @ W.t()).sub_(lse[:, None])).mul_(g64[:, None])
        t = owned(lo, W.shape[0])
        G[t, targets[t] - lo] -= g64[t]
        dH.addmm_(G, W)
        dW[p][r:r + W.shape[0]].addmm_(G.t(), H64)
    return {"loss": loss, "lse": lse, "dH": dH, "dW": dW}
