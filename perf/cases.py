"""The work that users have this package do, as cases that can be timed and compared.

An MoE instance runs `LayerStep.step_fused` (gating selection, activated-expert-balanced scheduling, dispatch,
grouped FFN, combine) once per layer and batch, so most cases are that call at the shapes of the repository's own
workloads, from a handful of requests to a chunk of thousands of tokens.  The others are the variants of that
call (gate inside the front launch, shared expert, fp32) and the two device calls of the control plane (batched
scheduling for the scaling model's a_max table, weight packing when a replica is pinned).

Inputs follow `paper_2512_13525_amd.workloads`: router logits N(0,1) plus the Zipf bias of the experts'
popularity, activations N(0,1), weights N(0, 0.02), a layout with the spare slots given to the hottest experts,
and, as the executed instance, the straggler of the batch (the one that sets the layer's latency).  The case's seed
draws the popularity ranking, the layout and all values."""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2512_13525_amd import binding as B
from paper_2512_13525_amd import workloads as W
from paper_2512_13525_amd.layer import LayerStep

# Layer dimensions, instances and replica slots of the repository's workloads, and one generic ragged shape: odd
# numbers of 32-column steps in both products (d_h, d_e multiples of 32 but not of 64), E no power of two.
MODELS = {
    "qwen3": dict(E=128, k=8, d_h=2048, d_e=768, n_inst=8, C=17, route="softmax", n_group=1, topk_group=1, zipf=1.0),
    "dsv2lite": dict(E=64, k=6, d_h=2048, d_e=1408, n_inst=4, C=17, route="softmax", n_group=1, topk_group=1, zipf=1.1),
    "dsv3": dict(E=256, k=8, d_h=7168, d_e=2048, n_inst=8, C=36, route="sigmoid_group", n_group=8, topk_group=4, zipf=1.2),
    "stress": dict(E=256, k=8, d_h=4096, d_e=1536, n_inst=16, C=16, route="softmax", n_group=1, topk_group=1, zipf=0.8),
    "ragged": dict(E=60, k=4, d_h=2016, d_e=1056, n_inst=3, C=22, route="softmax", n_group=1, topk_group=1, zipf=0.9),
    "tiny": dict(E=8, k=2, d_h=256, d_e=512, n_inst=2, C=5, route="softmax", n_group=1, topk_group=1, zipf=0.0),
}


def _case(name, kind, model, T, layers=1, dtype="bf16", d_s=0, batches=0, **kw):
    c = dict(name=name, kind=kind, T=T, layers=layers, dtype=dtype, d_s=d_s, batches=batches)
    c.update(MODELS[model])
    c.update(kw)
    return c


def listed():
    return [
        # A few requests in flight: the step's latency, launches and ramps.  Four layers a pass, each with weights of
        # its own, as a decode step walks them.
        _case("decode_qwen3_T8", "step", "qwen3", 8, layers=4),
        # Decode batches at the sizes the paper's instances run.
        _case("decode_qwen3_T256", "step", "qwen3", 256, layers=4),
        _case("decode_dsv2lite_T128", "step", "dsv2lite", 128, layers=4),
        _case("decode_dsv3_T512", "step", "dsv3", 512),
        # A batch between decode and prefill, odd number of tokens: tens to hundreds of rows per expert.
        _case("chunk_dsv2lite_T1000", "step", "dsv2lite", 1000),
        # A prefill chunk: the largest call.
        _case("chunk_stress_T8192", "step", "stress", 8192),
        # Ragged sizes in every dimension.
        _case("ragged_T203", "step", "ragged", 203, layers=4),
        # The instance receives activations and runs the gate itself (selection, schedule and dispatch from X).
        _case("gate_dsv3_T512", "gate", "dsv3", 512),
        # A model family with a shared expert that this instance runs too (width of one routed expert).
        _case("shared_dsv3_T256", "step", "dsv3", 256, d_s=2048),
        # The fp32 configuration, canonical weights.
        _case("f32_tiny_T64", "step", "tiny", 64, layers=4, dtype="f32"),
        # Monte-Carlo table of the scaling model: 2000 sampled batches scheduled in one call.
        _case("schedule_2000x256", "schedule", "stress", 256, batches=2000),
        # Weights of an instance packed when its replicas are pinned.
        _case("pack_dsv2lite", "pack", "dsv2lite", 0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Mostly layer steps of the workloads' shapes over the whole range of batch sizes, then ragged layer
    dimensions, then the variants.  Costs stay below the largest listed case (layers only for small batches)."""
    u = rng.random()
    if u < 0.55:
        model = rng.choice(["qwen3", "dsv2lite", "dsv3", "stress"])
        T = _log_int(rng, 1, {"qwen3": 4000, "dsv2lite": 3000, "dsv3": 512, "stress": 6000}[model])
        layers = 1 if model in ("dsv3", "stress") or T > 512 else rng.choice([1, 2, 4])
        zipf = round(rng.uniform(0.9 if model == "dsv3" else 0.0, 1.2), 2)
        d_s = MODELS[model]["d_e"] if rng.random() < 0.15 else 0
        return {k: v for k, v in _case("", "step", model, T, layers=layers, d_s=d_s, zipf=zipf).items() if k != "name"}
    if u < 0.75:
        n_inst = rng.choice([2, 3, 4, 6])
        E = n_inst * rng.randint(5, 24)
        c = _case("", "step", "ragged", _log_int(rng, 1, 1500), layers=rng.choice([1, 2]), E=E, n_inst=n_inst,
                  C=E // n_inst + rng.randint(0, 3), k=rng.randint(1, 8) if E >= 16 else 2,
                  d_h=32 * rng.randint(8, 80), d_e=32 * rng.randint(4, 50), zipf=round(rng.uniform(0.0, 1.2), 2))
    elif u < 0.85:
        model = rng.choice(["qwen3", "dsv2lite", "dsv3", "ragged"])
        c = _case("", "gate", model, _log_int(rng, 1, 1000))
    elif u < 0.9:
        c = _case("", "step", "tiny", _log_int(rng, 1, 300), layers=2, dtype="f32", d_h=4 * rng.randint(16, 160),
                  d_e=4 * rng.randint(16, 160))
    elif u < 0.95:
        c = _case("", "schedule", rng.choice(["stress", "qwen3", "dsv3"]), _log_int(rng, 16, 512),
                  batches=_log_int(rng, 100, 3000))
    else:
        c = _case("", "pack", "ragged", 0, C=rng.randint(4, 24), d_h=32 * rng.randint(16, 128), d_e=32 * rng.randint(8, 64))
    return {k: v for k, v in c.items() if k != "name"}


# ------------------------------------------------------------------ inputs
def _cfg(case, seed, layer=0):
    return W.MoEConfig("case", E=case["E"], k=case["k"], d_h=case["d_h"], d_e=case["d_e"], T=case["T"],
                       n_inst=case["n_inst"], C=case["C"], route=case["route"], n_group=case["n_group"],
                       topk_group=case["topk_group"], zipf_s=case["zipf"], dtype=case["dtype"], seed=1000 * seed + layer)


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _layout(cfg):
    if cfg.E == 8 and cfg.n_inst == 2 and cfg.C == 5:
        return np.array([0, 1, 2, 3, -1, 4, 5, 6, 7, 0], dtype=np.int32)
    return W.build_placement(cfg)


def _draw_normal(seed, stream, shape, scale, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1009 + stream) % (1 << 62))
    x = torch.empty(shape, dtype=dtype, device="cuda").normal_(generator=g)
    return x.mul_(scale) if scale != 1.0 else x


def _weights(case, cfg):
    C, d_h, d_e, dt = case["C"], case["d_h"], case["d_e"], _dtype(case)
    return (_draw_normal(cfg.seed, 1, (C, 2 * d_e, d_h), 0.02, dt), _draw_normal(cfg.seed, 2, (C, d_h, d_e), 0.02, dt))


def _shared_weights(case, cfg):
    return (_draw_normal(cfg.seed, 3, (2 * case["d_s"], case["d_h"]), 0.02, _dtype(case)),
            _draw_normal(cfg.seed, 4, (case["d_h"], case["d_s"]), 0.02, _dtype(case)))


def _activations(case, cfg):
    return _draw_normal(cfg.seed, 5, (case["T"], case["d_h"]), 1.0, _dtype(case))


def _router(case, cfg):
    bias = None
    if case["zipf"]:
        bias = torch.from_numpy(np.log(cfg.E * W.expert_popularity(cfg)).astype(np.float32)).cuda()
    return _draw_normal(cfg.seed, 6, (case["E"], case["d_h"]), case["d_h"] ** -0.5, _dtype(case)), bias


def _select(case, logits):
    """Top-k ids [T,k] and weights (64 bits) of the gating selection."""
    x = np.asarray(logits, dtype=np.float64)
    T, E = x.shape
    keep = x
    if case["route"] == "sigmoid_group":
        s = 1.0 / (1.0 + np.exp(-x))
        per = E // case["n_group"]
        score = np.sort(s.reshape(T, case["n_group"], per), axis=2)[:, :, -2:].sum(axis=2)
        best = np.argsort(-score, axis=1, kind="stable")[:, :case["topk_group"]]
        mask = np.zeros((T, case["n_group"]), dtype=bool)
        np.put_along_axis(mask, best, True, axis=1)
        keep = np.where(np.repeat(mask, per, axis=1), x, -np.inf)
    ids = np.argsort(-keep, axis=1, kind="stable")[:, :case["k"]]
    v = np.take_along_axis(x, ids, axis=1)
    w = 1.0 / (1.0 + np.exp(-v)) if case["route"] == "sigmoid_group" else np.exp(v - v.max(axis=1, keepdims=True))
    return ids, w / w.sum(axis=1, keepdims=True)


def _schedule(case, layout, ids):
    """Activated-expert-balanced scheduling: the instance and slot of every activated expert, and the loads."""
    n, C = case["n_inst"], case["C"]
    hosts = {}
    for rid, e in enumerate(layout):
        if e >= 0:
            hosts.setdefault(int(e), []).append(rid)
    act = np.unique(ids)
    load = np.zeros(n, dtype=np.int64)
    rep = np.full(case["E"], -1, dtype=np.int64)
    for single in (True, False):
        for e in act:
            rids = hosts[int(e)]
            if (len(rids) == 1) == single:
                r = min(rids, key=lambda q: (load[q // C], q // C))
                rep[e] = r
                load[r // C] += 1
    return rep, load


def _batch(case, seed, layer):
    cfg = _cfg(case, seed, layer)
    layout = _layout(cfg)
    logits = W.router_logits(cfg)
    ids, w = _select(case, logits)
    rep, load = _schedule(case, layout, ids)
    return cfg, layout, logits, ids, w, rep, int(np.argmax(load))


def _sampled_ids(case, cfg):
    """Top-k ids of `batches` sampled batches, from logits drawn on the GPU."""
    logits = _draw_normal(cfg.seed, 7, (case["batches"], case["T"], case["E"]), 1.0, torch.float32)
    if case["zipf"]:
        logits += torch.from_numpy(np.log(cfg.E * W.expert_popularity(cfg)).astype(np.float32)).cuda()
    return logits.topk(case["k"], dim=2).indices.to(torch.int32)


# ------------------------------------------------------------------ preparation and one pass
def prepare(case, seed):
    kind = case["kind"]
    if kind == "schedule":
        cfg = _cfg(case, seed)
        pl = B.Placement(_layout(cfg), cfg.E, cfg.n_inst, cfg.C)
        return dict(case=case, pl=pl, ids=_sampled_ids(case, cfg).contiguous(),
                    load=torch.empty((case["batches"], cfg.n_inst), dtype=torch.int32, device="cuda"))
    if kind == "pack":
        W13, W2 = _weights(case, _cfg(case, seed))
        return dict(case=case, W13=W13, W2=W2, W13p=torch.empty_like(W13), W2p=torch.empty_like(W2))
    if kind == "gate":
        cfg = _cfg(case, seed)
        Wr, bias = _router(case, cfg)
        return dict(case=case, step=LayerStep(cfg, _layout(cfg), 0), X=_activations(case, cfg), Wr=Wr, bias=bias)
    layers = []
    for layer in range(case["layers"]):
        cfg, layout, logits, _, _, _, g = _batch(case, seed, layer)
        step = LayerStep(cfg, layout, g)
        step.set_weights(*_weights(case, cfg))
        if case["d_s"]:
            step.enable_shared(*_shared_weights(case, cfg))
        layers.append((step, torch.from_numpy(logits).cuda(), _activations(case, cfg)))
    return dict(case=case, layers=layers)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "schedule":
        B.moe_schedule_batched(state["pl"], state["ids"], case["batches"], case["T"], case["k"], None, None, state["load"])
        return state["load"]
    if kind == "pack":
        B.moe_pack_weights_bf16(state["W13"], state["W2"], case["C"], case["d_h"], case["d_e"], state["W13p"], state["W2p"])
        return [state["W13p"], state["W2p"]]
    if kind == "gate":
        s = state["step"]
        logits = s.front_gate(state["X"], state["Wr"], state["bias"])
        return dict(logits=logits, ids=s.topk_ids, w=s.topk_w, rid=s.rid, load=s.load, count=s.slot_count)
    out = []
    for step, logits, X in state["layers"]:
        Y = step.step_fused_shared(logits, X) if case["d_s"] else step.step_fused(logits, X)
        out.append(dict(Y=Y, ids=step.topk_ids, w=step.topk_w, rid=step.rid, load=step.load, count=step.slot_count))
    return out


# ------------------------------------------------------------------ what a pass cannot do without, and how exact it is
def work(case):
    kind, T, k, E = case["kind"], case["T"], case["k"], case["E"]
    size = 2 if case["dtype"] == "bf16" else 4
    if kind == "schedule":
        return {"bytes": 4 * case["batches"] * (T * k + case["n_inst"]), "flops": 0}
    if kind == "pack":
        return {"bytes": 2 * 2 * 3 * case["C"] * case["d_h"] * case["d_e"], "flops": 0}
    if kind == "gate":
        return {"bytes": 2 * (T + E) * case["d_h"] + 4 * T * E + 3 * 4 * T * k, "flops": 2 * T * E * case["d_h"]}
    moved = flops = 0
    for layer in range(case["layers"]):
        _, _, _, ids, _, rep, g = _batch(case, 0, layer)
        slots = rep[ids]
        local = (slots >= g * case["C"]) & (slots < (g + 1) * case["C"])
        expert = 3 * case["d_h"] * case["d_e"]
        moved += len(np.unique(slots[local])) * expert * size              # weights of the activated experts
        rows = T if case["d_s"] else int(local.any(axis=1).sum())
        moved += rows * case["d_h"] * size + T * case["d_h"] * size        # token rows in, output rows out
        moved += 4 * T * E + 3 * 4 * T * k                                 # logits in; ids, weights, replica ids out
        flops += 2 * expert * int(local.sum())
        if case["d_s"]:
            moved += 3 * case["d_h"] * case["d_s"] * size
            flops += 2 * 3 * case["d_h"] * case["d_s"] * T
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    # About four times the relative error measured against exact(): bf16 steps 2.3e-3 .. 2.5e-3 (2^-9 of rounding in the
    # intermediate and again in the result; largest single difference 4e-2), fp32 steps 1.6e-7 (largest 1e-6), router
    # logits of the gate 1.1e-7 (largest 4e-7); fp32 sums in another order stay within 1e-6.
    if case["kind"] in ("schedule", "pack"):
        return "exact"
    if case["kind"] == "gate":
        # logits closer together than their rounding may change places in the selection
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-3}
    return {"rel": 1e-2, "max": 0.1} if case["dtype"] == "bf16" else {"rel": 1e-6, "max": 1e-5}


def _ffn64(X, W13, W2):
    d_e = W2.shape[1]
    h = X.double() @ W13.double().t()
    g, u = h[:, :d_e], h[:, d_e:]
    return (g / (1.0 + torch.exp(-g)) * u) @ W2.double().t()


def exact(case, seed):
    kind = case["kind"]
    if kind in ("schedule", "pack"):                                       # whole numbers, moved bytes
        return None
    if kind == "gate":
        cfg = _cfg(case, seed)
        Wr, bias = _router(case, cfg)
        logits = _activations(case, cfg).double() @ Wr.double().t()
        if bias is not None:
            logits += bias.double()
        _, w = _select(case, logits.cpu().numpy())
        return dict(logits=logits, ids=None, w=torch.from_numpy(w), rid=None, load=None, count=None)
    out = []
    for layer in range(case["layers"]):
        cfg, _, _, ids, w, rep, g = _batch(case, seed, layer)
        W13, W2 = _weights(case, cfg)
        X = _activations(case, cfg)
        Y = torch.zeros((case["T"], case["d_h"]), dtype=torch.float64, device="cuda")
        slots = rep[ids] - g * case["C"]
        for s in np.unique(slots[(slots >= 0) & (slots < case["C"])]):
            tok, choice = np.nonzero(slots == s)
            t = torch.from_numpy(tok).cuda()
            wt = torch.from_numpy(w[tok, choice]).cuda()
            Y.index_add_(0, t, _ffn64(X[t], W13[int(s)], W2[int(s)]) * wt[:, None])
        if case["d_s"]:
            Y += _ffn64(X, *_shared_weights(case, cfg))
        out.append(dict(Y=Y, ids=None, w=torch.from_numpy(w), rid=None, load=None, count=None))
    return out
