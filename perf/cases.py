"""The calls this library is measured on, over the range its users run.

The layer shapes are those of the models the paper evaluates (a Mixtral-8x7B-, a Qwen2-57B-A14B- and a
Qwen1.5-MoE-A2.7B-shaped layer) and the small fp32 layer of the parity tests; `draw` adds generic shapes.  Inputs are
drawn on the GPU from the seed alone: x ~ N(0, 1), weights ~ N(0, 0.02), router logits ~ N(0, 1) plus a per-expert bias.

Paths (`case["path"]`):
  forward    one masked layer forward on the ranked weights, optionally right after a budget switch
  noalloc    the forward that takes no workspace (serving loops that must not allocate)
  clipped    the forward on one budget's exported compact weights
  saliency   one calibration batch of the channel ranking: scores cleared, then accumulated
  action     one action-learning step: sampled widths, forward, backward, action gradient
  rank       the one-time preparation of a layer: rank and reorder its channels, export one budget
"""
import math

import numpy as np
import torch

from paper_2606_27866_amd import flexmoe as fm

QWEN2 = dict(d=3584, E=64, I=2560, top_k=8, I_shared=20480, norm=0)
QWEN15 = dict(d=2048, E=60, I=1408, top_k=4, I_shared=5632, norm=0)
MIXTRAL = dict(d=4096, E=8, I=14336, top_k=2, I_shared=0, norm=1)
TINY = dict(d=256, E=8, I=512, top_k=2, I_shared=0, norm=1)
RATIOS = (0.1, 0.4, 0.7, 1.0)  # retention ratios an expert chooses from


def _case(name, shape, path, T, dtype="bf16", kept=0.5, widths="grid", skew=False, switch=False):
    c = dict(shape, path=path, T=T, dtype=dtype, kept=kept, widths=widths, skew=skew, switch=switch)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: the fp32 layer of the parity tests, all latency and launches
        _case("tiny_f32_T64", TINY, "forward", 64, dtype="f32", kept=0.6, widths="odd"),
        # fp32 at a real layer's size: checking a bf16 deployment against full precision
        _case("qwen15_f32_T500", QWEN15, "forward", 500, dtype="f32", kept=0.5),
        # one user's decode step, the budget changed for this step (online clipping)
        _case("qwen2_decode_T1", QWEN2, "forward", 1, kept=0.6, switch=True),
        # a decode batch of a server, widths as action learning leaves them (multiples of nothing)
        _case("qwen2_decode_T24", QWEN2, "forward", 24, kept=0.6, widths="actions"),
        # a decode batch inside a captured or allocation-free serving loop
        _case("qwen15_noalloc_T37", QWEN15, "noalloc", 37, kept=0.8),
        # a large decode batch or a chunk of a chunked prefill
        _case("qwen2_T300", QWEN2, "forward", 300, kept=0.6, widths="actions"),
        # one prompt on an offline-clipped checkpoint
        _case("qwen15_clipped_T1023", QWEN15, "clipped", 1023, kept=0.4),
        # a prefill batch with a shared expert
        _case("qwen2_prefill_T8192", QWEN2, "forward", 8192, kept=0.6),
        # the headline: a large prefill batch over few wide experts with skewed load
        _case("mixtral_prefill_T16384", MIXTRAL, "forward", 16384, kept=0.5, skew=True),
        # one calibration batch of the channel ranking
        _case("qwen15_saliency_T4096", QWEN15, "saliency", 4096, kept=1.0),
        # one action-learning step
        _case("qwen15_action_T4096", QWEN15, "action", 4096, kept=0.5),
        # ranking, reorder and export of one layer before deployment
        _case("qwen15_rank", QWEN15, "rank", 0, kept=0.5),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choice(["forward"] * 5 + ["noalloc", "clipped", "saliency", "action", "rank"])
    dtype = "f32" if path in ("forward", "rank", "clipped") and rng.random() < 0.2 else "bf16"
    if rng.random() < 0.6:
        shape = dict(rng.choice([QWEN2, QWEN15, MIXTRAL]))
    else:
        E = rng.randint(4, 96)
        shape = dict(d=8 * log_int(32, 512), E=E, I=8 * log_int(16, 512), top_k=rng.randint(1, min(E, 10)),
                     I_shared=rng.choice([0, 8 * log_int(64, 1024)]), norm=rng.randint(0, 1))
    if dtype == "f32" and shape["d"] > 2048:
        shape["E"] = min(shape["E"], 8)
        shape["top_k"] = min(shape["top_k"], 4)
    lo, hi = {"forward": (1, 16384), "clipped": (1, 8192), "noalloc": (1, 64), "saliency": (256, 8192),
              "action": (256, 8192), "rank": (1, 1)}[path]
    if dtype == "f32":
        hi = min(hi, 1024)
    T = 0 if path == "rank" else log_int(lo, hi)
    c = _case("", shape, path, T, dtype, kept=1.0 if path == "saliency" else rng.choice([0.2, 0.4, 0.6, 0.8, 1.0]),
              widths=rng.choice(["grid", "actions", "odd"]), skew=rng.random() < 0.3,
              switch=path == "forward" and rng.random() < 0.3)
    most = max(work(x)["flops"] for x in listed())
    scale = 16 if dtype == "f32" else 1.6 if path in ("saliency", "action") else 1  # such work runs at a lower rate
    while work(c)["flops"] * scale > most:
        c["T"] = max(1, c["T"] * 2 // 3)
    return c


# ---- inputs -----------------------------------------------------------------
def _widths(case, seed):
    """Per-expert keep counts of about case["kept"] of the routed channels."""
    E, I = case["E"], case["I"]
    # a deployment exports the budget it was given: the same one for every layer's weights
    rng = np.random.Generator(np.random.PCG64(7000 + (0 if case["path"] == "rank" else seed)))
    k = np.full(E, I, np.int64)
    want = case["kept"] * E * I
    if case["widths"] == "grid":      # nested budgets: 64-channel steps removed at random, down to nothing
        while k.sum() > want:
            e = rng.integers(E)
            k[e] -= min(64, k[e])
    elif case["widths"] == "actions":  # one retention ratio per expert
        level = np.full(E, len(RATIOS) - 1)
        while k.sum() > want and level.max() > 0:
            e = rng.integers(E)
            level[e] = max(level[e] - 1, 0)
            k[e] = math.ceil(RATIOS[level[e]] * I - 1e-9)
    else:                              # any width
        k = np.clip(np.round(case["kept"] * I * rng.uniform(0.5, 1.5, E)), 0, I).astype(np.int64)
    return k.astype(np.int32)


def _inputs(case, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(1234567 + seed)
    td = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    d, E, I, Is, T = case["d"], case["E"], case["I"], case["I_shared"], case["T"]

    def normal(*shape, std=1.0, dtype=td):
        out = torch.empty(shape, dtype=dtype, device=dev)
        return out.normal_(0.0, std, generator=g)

    bias = normal(E, std=0.5, dtype=torch.float32)
    if case["skew"]:  # a few popular experts: about a Zipf(1.2) load
        rank = torch.randperm(E, generator=g, device=dev).float() + 1.0
        bias = -0.9 * torch.log(rank)
    return dict(
        x=normal(T, d), logits=normal(T, E, dtype=torch.float32) + bias,
        w=[normal(E, I, d, std=0.02), normal(E, I, d, std=0.02), normal(E, d, I, std=0.02)],
        ws=[normal(Is, d, std=0.02), normal(Is, d, std=0.02), normal(d, Is, std=0.02)] if Is else [None] * 3,
        keep=_widths(case, seed),
        target=normal(T, d, std=0.05, dtype=torch.float32) if case["path"] == "saliency" else None,
        dy=normal(T, d, std=1e-3, dtype=torch.float32) if case["path"] == "action" else None,
        alpha=normal(E, len(RATIOS), dtype=torch.float32),
        gumbel=-torch.log(-torch.log(torch.rand(E, len(RATIOS), generator=g, device=dev).clamp_(1e-7, 1 - 1e-6))),
        scores=normal(E, I, dtype=torch.float32).square_() if case["path"] == "rank" else None)


TAU, LAMBDA, BETA = 1.0, 1e-3, 1e-3


def prepare(case, seed):
    inp = _inputs(case, seed)
    dt = fm.FLEXMOE_BF16 if case["dtype"] == "bf16" else fm.FLEXMOE_F32
    T = max(case["T"], 1)
    layer = fm.Layer(case["d"], case["E"], case["I"], case["top_k"], case["I_shared"], dt, case["norm"], max_tokens=T)
    layer.set_weights(*inp["w"], *inp["ws"])
    layer.set_budget(inp["keep"])
    st = dict(inp, path=case["path"], T=case["T"], switch=case["switch"], layer=layer)
    if case["path"] == "clipped":
        st["clipped"] = layer.export_clipped(inp["keep"])
    elif case["path"] == "noalloc":
        st["y"] = torch.empty_like(inp["x"])
    elif case["path"] == "saliency":
        st["saliency"] = fm.Saliency(layer, T)
    elif case["path"] == "action":
        st["learner"] = fm.ActionLearner(layer, T, RATIOS)
        st["learner"].transpose_weights()
    return st


def run(state):
    layer, path = state["layer"], state["path"]
    if path == "forward":
        if state["switch"]:
            layer.set_budget(state["keep"])
        return layer.forward(state["x"], state["logits"])
    if path == "clipped":
        return layer.forward(state["x"], state["logits"], clipped=state["clipped"])
    if path == "noalloc":
        fm.flexmoe_layer_forward_noalloc(layer.desc, state["T"], state["x"], state["logits"], layer.w_gate, layer.w_up,
                                         layer.w_down, layer.keep, layer.ws_gate, layer.ws_up, layer.ws_down,
                                         state["y"])
        return state["y"]
    if path == "saliency":
        sal = state["saliency"]
        sal.scores.zero_()
        sal.add_batch(state["x"], state["logits"], state["target"])
        return sal.scores
    if path == "rank":
        gate, up, down, perm = _rank(layer, state["scores"])
        ranked = fm.Layer.__new__(fm.Layer)
        ranked.__dict__.update(layer.__dict__)
        ranked.set_weights(gate, up, down, *state["ws"])
        c = ranked.export_clipped(state["keep"])
        n = c.packed_channels * layer.desc.d
        return {"gate": gate, "up": up, "down": down, "perm": perm, "gate_c": c.w_gate_c[:n], "up_c": c.w_up_c[:n],
                "down_c": c.w_down_c[:n]}
    learner = state["learner"]
    learner.sample(state["alpha"], state["gumbel"])
    y = learner.forward(state["x"], state["logits"])
    dx, dl, dm = learner.backward(state["logits"], state["dy"])
    da, stats = learner.action_grad(state["alpha"], state["gumbel"], TAU, LAMBDA, BETA, dm)
    return {"keep": learner.keep, "y": y, "dx": dx, "dlogits": dl, "dmask": dm, "dalpha": da, "stats": stats}


def _rank(layer, scores):
    out = [torch.empty_like(w) for w in (layer.w_gate, layer.w_up, layer.w_down)]
    perm = torch.empty((layer.desc.E, layer.desc.I), dtype=torch.int32, device=scores.device)
    fm.flexmoe_rank_reorder(layer.desc, scores, layer.w_gate, layer.w_up, layer.w_down, *out, perm)
    return (*out, perm)


# ---- what a pass cannot do without ------------------------------------------
def work(case):
    d, E, I, k, Is, T = (case[n] for n in ("d", "E", "I", "top_k", "I_shared", "T"))
    es = 2 if case["dtype"] == "bf16" else 4
    f = case["kept"]
    if case["path"] == "rank":
        return {"bytes": 6 * E * I * d * es + 8 * E * I + 6 * f * E * I * d * es, "flops": 0}
    # experts that some token reaches, under about the load the router biases give
    load = np.arange(1, E + 1) ** -0.9 if case["skew"] else np.exp(0.5 * np.linspace(-2, 2, E))
    active = float(np.sum(1 - (1 - np.minimum(1, k * load / load.sum())) ** T))
    rows = T * k
    io = 2 * T * d * es + 4 * T * E
    if case["path"] == "saliency":
        return {"bytes": 3 * d * es * (active * I + Is) + io + 4 * T * d + 4 * E * I,
                "flops": 14 * d * rows * I + 6 * d * T * Is}
    if case["path"] == "action":
        f = sum(RATIOS) / len(RATIOS)
        return {"bytes": 3 * d * es * (active * I + Is) + io + 12 * T * d + 4 * T * E + 4 * E * I,
                "flops": d * rows * I * (6 + 6 * f) + 12 * d * T * Is}
    return {"bytes": 3 * d * es * (active * f * I + Is) + io, "flops": 6 * d * (f * rows * I + T * Is)}


def tolerance(case):
    if case["path"] == "rank":
        return "exact"  # sorted and copied, nothing is computed
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["path"] == "saliency":
        return {"rel": 2e-2}  # sums of squares of gradients of bf16 activations
    if case["path"] == "action":
        return {"rel": 1e-2}
    # bf16 results, with the activations and each expert's output rounded to bf16 on the way
    return {"rel": 1e-2}


# ---- the same results in 64 bits --------------------------------------------
def _route(logits, k, norm):
    p = torch.softmax(logits, dim=1)
    idx = torch.sort(logits, dim=1, descending=True, stable=True).indices[:, :k]
    w = p.gather(1, idx)
    if norm:
        w = w / w.sum(1, keepdim=True)
    return idx, w


def _segments(idx, E):
    """(tokens, slots) of every expert."""
    for e in range(E):
        t, j = torch.nonzero(idx == e, as_tuple=True)
        yield e, t, j


def exact(case, seed):
    inp = _inputs(case, seed)
    D = torch.float64
    E, I, k, T, d = case["E"], case["I"], case["top_k"], case["T"], case["d"]
    keep = inp["keep"].astype(np.int64)
    if case["path"] == "rank":
        return _exact_rank(case, inp, keep)
    if case["path"] == "action":
        act = torch.argmax(inp["alpha"] + inp["gumbel"], dim=1).cpu().numpy()
        keep = np.array([max(1, math.ceil(RATIOS[a] * I - 1e-9)) for a in act], np.int64)
    elif case["path"] == "saliency":
        keep = np.full(E, I, np.int64)
    x = inp["x"].to(D)
    lg = inp["logits"].to(D).requires_grad_(case["path"] == "action")
    idx, w = _route(lg, k, case["norm"])
    wd_ = w.detach()
    W = inp["w"]
    y = torch.zeros((T, d), dtype=D, device=x.device)
    silu = torch.nn.functional.silu
    for e, t, j in _segments(idx, E):
        n = int(keep[e])
        if n == 0 or t.numel() == 0:
            continue
        h = silu(x[t] @ W[0][e, :n].to(D).T) * (x[t] @ W[1][e, :n].to(D).T)
        y.index_add_(0, t, wd_[t, j].unsqueeze(1) * (h @ W[2][e, :, :n].to(D).T))
    s64 = [s.to(D) for s in inp["ws"]] if case["I_shared"] else None
    if s64:
        gs, us = x @ s64[0].T, x @ s64[1].T
        y += (silu(gs) * us) @ s64[2].T
    if case["path"] not in ("saliency", "action"):
        return y

    dY = y - inp["target"].to(D) if case["path"] == "saliency" else inp["dy"].to(D)
    scores = torch.zeros((E, I), dtype=D, device=x.device)
    dx = torch.zeros_like(x)
    dmask = torch.zeros((E, I), dtype=D, device=x.device)
    dw = torch.zeros_like(wd_)
    for e, t, j in _segments(idx, E):
        if t.numel() == 0:
            continue
        n = int(keep[e])
        wg, wu, wn = W[0][e].to(D), W[1][e].to(D), W[2][e].to(D)
        xe = x[t]
        g, u = xe @ wg.T, xe @ wu.T
        sg = torch.sigmoid(g)
        a = g * sg
        dO = wd_[t, j].unsqueeze(1) * dY[t]
        dh = dO @ wn
        dG, dU = dh * u * (sg * (1 + g * (1 - sg))), dh * a
        if case["path"] == "saliency":
            scores[e] = (wg * (dG.T @ xe)).square().sum(1) + (wu * (dU.T @ xe)).square().sum(1)
            scores[e] += (wn * (dO.T @ (a * u))).square().sum(0)
            continue
        dmask[e] = (dh * a * u).sum(0)
        dw[t, j] = (dY[t] * ((a * u)[:, :n] @ wn[:, :n].T)).sum(1)
        dx.index_add_(0, t, dG[:, :n] @ wg[:n] + dU[:, :n] @ wu[:n])
    if case["path"] == "saliency":
        return scores
    if s64:
        sg = torch.sigmoid(gs)
        dh = dY @ s64[2]
        dx += (dh * us * (sg * (1 + gs * (1 - sg)))) @ s64[0] + (dh * gs * sg) @ s64[1]
    w.backward(dw)
    da, stats = _exact_actions(case, inp, idx, dmask)
    return {"keep": None, "y": y, "dx": dx, "dlogits": lg.grad, "dmask": dmask, "dalpha": da, "stats": stats}


def _exact_actions(case, inp, idx, dmask):
    D = torch.float64
    E, I = case["E"], case["I"]
    r = torch.tensor(RATIOS, dtype=D, device=dmask.device)
    wid = [max(1, math.ceil(q * I - 1e-9)) for q in RATIOS]
    z = torch.softmax((inp["alpha"].to(D) + inp["gumbel"].to(D)) / TAU, dim=1)
    dz = torch.stack([dmask[:, :n].sum(1) for n in wid], dim=1)
    p = torch.softmax(inp["alpha"].to(D), dim=1)
    H = -(p * p.log()).sum(1, keepdim=True)
    q = torch.bincount(idx.reshape(-1), minlength=E).to(D).unsqueeze(1) / idx.numel()
    pr = (p * r).sum(1, keepdim=True)
    da = z * (dz - (z * dz).sum(1, keepdim=True)) / TAU
    da += LAMBDA * q * p * (r - pr) + BETA * p * (p.log() + H) / E
    return da, torch.stack([(q * pr).sum(), H.mean()])


def _exact_rank(case, inp, keep):
    perm = torch.sort(inp["scores"], dim=1, descending=True, stable=True).indices
    gate, up, down = inp["w"]
    E, d = case["E"], case["d"]
    out = {"gate": torch.stack([gate[e][perm[e]] for e in range(E)]),
           "up": torch.stack([up[e][perm[e]] for e in range(E)]),
           "down": torch.stack([down[e][:, perm[e]] for e in range(E)])}

    def packed(e, n):
        return (int(n) + 7) // 8 * 8

    for name in ("gate", "up", "down"):
        rows = []
        for e in range(E):
            blk = out[name][e].T if name == "down" else out[name][e]
            b = torch.zeros((packed(e, keep[e]), d), dtype=blk.dtype, device=blk.device)
            b[:keep[e]] = blk[:keep[e]]
            rows.append((b.T if name == "down" else b).reshape(-1))
        out[name + "_c"] = torch.cat(rows)
    return {"gate": out["gate"], "up": out["up"], "down": out["down"], "perm": None, "gate_c": out["gate_c"],
            "up_c": out["up_c"], "down_c": out["down_c"]}
