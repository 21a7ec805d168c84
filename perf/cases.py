"""The work that a program has the expert layer do, as cases to be timed.

Four kinds of call, through the package's entry points:

* "forward"  LLEPLayer.forward over every virtual device (device -1);
* "share"    LLEPLayer.forward of the most-loaded virtual device's groups
             alone (what one rank of an expert-parallel job computes);
* "train"    forward that keeps g and u, then LLEPLayer.backward, over every
             virtual device: y, input, gate and weight gradients;
* "pack"     llep_pack_weights and llep_pack_weights_backward, which a
             training program runs after every update of its weights.

Sizes are those of the layer configurations in synth.py (their hidden and
FFN sizes, experts, top-k, capacity factor and routing skew) with token
counts from one decoded token to those configurations' full batches; drawn
cases also take generic layer sizes.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2601_17111_amd import binding as B
from paper_2601_17111_amd import synth
from paper_2601_17111_amd.layer import LLEPLayer

# hidden size, FFN size, experts, experts per token, capacity factor
SHAPES = {
    "tiny": (64, 128, 8, 2, 1.25),
    "gpt-oss-20b": (2880, 2880, 32, 4, 1.1),
    "gpt-oss-120b": (2880, 2880, 128, 4, 1.1),
    "qwen3-30b-a3b": (2048, 768, 128, 8, 1.1),
    "deepseek-v3": (7168, 2048, 256, 8, 1.0),
}


def _case(kind, T, shape, routing, a, b, *, mode="llep", dtype="bf16", P=8):
    """routing "hot": a of the pairs on b experts; "zipf": exponent a."""
    D, F, E, K, alpha = SHAPES[shape] if isinstance(shape, str) else shape
    return {"kind": kind, "T": T, "D": D, "F": F, "E": E, "K": K, "P": P, "alpha": alpha,
            "routing": routing, "a": a, "b": b, "mode": mode, "dtype": dtype}


def listed():
    cases = {
        # one token of one stream: latency, launches and the weights of K experts
        "decode-1-gpt-oss-20b": _case("forward", 1, "gpt-oss-20b", "hot", 0.6, 4),
        # decode of a small batch with an odd count; skewed routing
        "decode-37-qwen3-30b-a3b": _case("forward", 37, "qwen3-30b-a3b", "zipf", 1.2, 0),
        # decode batch with one dominating expert and many experts of one row
        "decode-64-deepseek-v3": _case("forward", 64, "deepseek-v3", "hot", 0.95, 1),
        # a full serving batch: every expert has a few rows
        "decode-256-gpt-oss-120b": _case("forward", 256, "gpt-oss-120b", "hot", 0.8, 4),
        # a ragged prompt under the standard expert-parallel plan
        "prefill-1001-qwen3-30b-a3b": _case("forward", 1001, "qwen3-30b-a3b", "zipf", 1.2, 0,
                                            mode="ep"),
        # an ordinary prefill batch
        "prefill-4096-gpt-oss-20b": _case("forward", 4096, "gpt-oss-20b", "hot", 0.6, 4),
        # one rank's share of the full batch, all skew on one expert
        "share-32768-gpt-oss-120b": _case("share", 32768, "gpt-oss-120b", "hot", 0.8, 1),
        # the same beside many nearly empty native experts
        "share-8192-deepseek-v3": _case("share", 8192, "deepseek-v3", "hot", 0.95, 1),
        # training steps of a layer: large experts, and many small ones
        "train-2048-gpt-oss-20b": _case("train", 2048, "gpt-oss-20b", "hot", 0.6, 4),
        "train-8192-qwen3-30b-a3b": _case("train", 8192, "qwen3-30b-a3b", "zipf", 1.2, 0),
        # the float32 layer at its reference configuration
        "train-256-tiny-f32": _case("train", 256, "tiny", "hot", 0.35, 1, dtype="f32", P=4),
        # re-packing after a weight update
        "pack-gpt-oss-20b": _case("pack", 1, "gpt-oss-20b", "hot", 0.6, 4),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    w = work(case)
    return w["bytes"] / 5e12 + w["flops"] / 1e15


def draw(rng):
    case = _draw(rng)
    most = max(_cost(c) for c in listed())
    while case["T"] > 1 and _cost(case) > most:
        case["T"] = max(1, case["T"] * 3 // 4)
    return case


def _draw(rng):
    kind = rng.choice(["decode"] * 5 + ["prefill"] * 4 + ["share"] * 2 + ["train"] * 3
                      + ["f32"] * 2 + ["pack"])
    # a layer of the repository's configurations, or a generic one
    shape = rng.choice(["gpt-oss-20b", "gpt-oss-120b", "qwen3-30b-a3b", "deepseek-v3", None, None])
    if kind in ("train", "pack") and shape in ("gpt-oss-120b", "deepseek-v3"):
        shape = None  # their float32 weight gradients alone fill much of a card
    if kind == "prefill" and shape == "deepseek-v3":
        shape = "qwen3-30b-a3b"  # a rank holds its share of that layer, not all of it
    if shape is None:
        shape = (64 * rng.randint(8, 64), 64 * rng.randint(6, 40),
                 rng.choice([16, 32] if kind in ("train", "pack") else [16, 32, 64]),
                 rng.choice([1, 2, 4, 6, 8]), rng.choice([1.0, 1.1, 1.25]))
    if rng.random() < 0.5:
        routing, a, b = "hot", round(rng.uniform(0.1, 0.95), 2), rng.choice([1, 4, 16])
    else:
        routing, a, b = "zipf", round(rng.uniform(0.0, 1.5), 2), 0
    mode = rng.choice(["llep", "llep", "ep"])
    if kind == "decode":
        return _case("forward", _log_int(rng, 1, 512), shape, routing, a, b, mode=mode,
                     P=rng.choice([1, 4, 8]))
    if kind == "prefill":
        return _case("forward", _log_int(rng, 512, 8192), shape, routing, a, b, mode=mode,
                     P=rng.choice([1, 4, 8]))
    if kind == "share":
        return _case("share", _log_int(rng, 4096, 32768), shape, routing, a, b)
    if kind == "train":
        return _case("train", _log_int(rng, 128, 8192), shape, routing, a, b, mode=mode)
    if kind == "f32":
        shape = (64 * rng.randint(1, 8), 64 * rng.randint(1, 8), rng.choice([8, 16]),
                 rng.choice([1, 2, 4]), 1.25)
        return _case(rng.choice(["forward", "train"]), _log_int(rng, 16, 768), shape, "hot",
                     round(rng.uniform(0.1, 0.9), 2), 1, mode=mode, dtype="f32", P=4)
    return _case("pack", 1, shape, routing, a, b)


# ---- inputs -------------------------------------------------------------------

def _dt(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _capacity(case):
    return int(math.ceil(case["alpha"] * case["T"] * case["K"] / case["P"] - 1e-9))


def _ids(case, seed):
    """Routing ids [T, K] and gates (softmax over K) as numpy arrays."""
    routing = (("hot", case["a"], case["b"]) if case["routing"] == "hot" else ("zipf", case["a"]))
    cfg = synth.LayerConfig("case", case["T"], case["D"], case["F"], case["E"], case["K"],
                            case["P"], 1, case["dtype"], routing)
    rng = np.random.default_rng([seed, 1])
    return synth.draw_ids(cfg, rng), synth.draw_gates(cfg, rng)


def _inputs(case, seed):
    ids, gates = _ids(case, seed)
    T, D, F, E = case["T"], case["D"], case["F"], case["E"]
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * seed + 17)

    def normal(*shape, std=1.0):
        return torch.empty(shape, dtype=_dt(case), device="cuda").normal_(0.0, std, generator=g)

    return dict(ids=torch.from_numpy(ids).cuda(), gates=torch.from_numpy(gates).cuda(),
                x=normal(T, D), dy=normal(T, D) if case["kind"] == "train" else None,
                w_gate=normal(E, D, F, std=0.02), w_up=normal(E, D, F, std=0.02),
                w_down=normal(E, F, D, std=0.02))


def prepare(case, seed):
    s = _inputs(case, seed)
    s["kind"] = case["kind"]
    raw = s["w_gate"], s["w_up"], s["w_down"]
    if case["kind"] == "pack":
        return s
    # the weights as the layer reads them; a program keeps the packed copies
    s["w_gate_up"], s["w_down_p"] = B.llep_pack_weights(*raw)
    if case["kind"] == "train":
        s["w_gate_up_t"], s["w_down_t"] = B.llep_pack_weights_backward(*raw)
    del s["w_gate"], s["w_up"], s["w_down"], raw
    layer = LLEPLayer(case["T"], case["K"], case["E"], case["P"], case["D"], case["F"],
                      _capacity(case), _dt(case), mode=case["mode"])
    s["layer"], s["device"] = layer, -1
    if case["kind"] == "share":
        # the rank that this process is; the other ranks' rows are not here
        layer.plan(s["ids"])
        s["device"] = layer.bufs.info_dict()["max_device"]
        layer.out_perm.zero_()
    return s


def run(s):
    if s["kind"] == "pack":
        raw = s["w_gate"], s["w_up"], s["w_down"]
        return B.llep_pack_weights(*raw) + B.llep_pack_weights_backward(*raw)
    layer = s["layer"]
    if s["kind"] != "train":
        return layer.forward(s["ids"], s["gates"], s["x"], s["w_gate_up"], s["w_down_p"],
                             device=s["device"])
    y = layer.forward(s["ids"], s["gates"], s["x"], s["w_gate_up"], s["w_down_p"],
                      save_gate_up=True)
    return (y,) + layer.backward(s["dy"], s["gates"], s["w_gate_up"], s["w_gate_up_t"],
                                 s["w_down_t"])


# ---- what a pass cannot do without -----------------------------------------------

def work(case):
    T, D, F, E, K = (case[k] for k in ("T", "D", "F", "E", "K"))
    eb = 2 if case["dtype"] == "bf16" else 4
    mat = 3 * D * F  # one expert's weights
    if case["kind"] == "pack":  # raw weights read once, both packed forms written
        return {"bytes": 3.0 * E * mat * eb, "flops": 0.0}
    ids, _ = _ids(case, 0)
    rows, experts = T * K, len(np.unique(ids))
    if case["kind"] == "share":
        on = _pairs_of(case, ids)[1]
        rows, experts = int(on.sum()), len(np.unique(ids.reshape(-1)[on]))
    # ids and gates, x in, y out, the weights of the experts in use
    nbytes = 8.0 * T * K + 2.0 * T * D * eb + experts * mat * eb
    flops = 2.0 * mat * rows
    if case["kind"] == "train":
        # dy in, dx and d gates out, the backward's weights in, float32 weight gradients out
        nbytes += 2.0 * T * D * eb + 4.0 * T * K + experts * mat * eb + E * mat * 4
        flops *= 3
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "pack":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 4e-4}
    return {"rel": 1e-2, "max": 0.2}


# ---- the same in 64 bits ------------------------------------------------------------

def _plan_share(case, loads):
    """Rows [start, end) of each expert that each device computes, as a list
    of (device, expert, start, end): the least-loaded assignment with chunks
    of any size, or standard expert parallelism."""
    E, P, cap = case["E"], case["P"], _capacity(case)
    M = E // P
    if case["mode"] == "ep" or P == 1:
        return [(e // M, e, 0, int(loads[e])) for e in range(E) if loads[e]]
    total = [int(loads[d * M:(d + 1) * M].sum()) for d in range(P)]
    chunks = []
    for e in sorted(range(E), key=lambda i: (-loads[i], i)):
        left, d = int(loads[e]), e // M
        if left == 0:
            continue
        keep = min(left, max(0, cap - (total[d] - left)))
        total[d] -= left - keep
        if keep:
            chunks.append((d, e, 0, keep))
        at, left = keep, left - keep
        while left:
            o = min((i for i in range(P) if i != d), key=lambda i: (total[i], i))
            n = min(left, cap - total[o]) if cap > total[o] else left
            chunks.append((o, e, at, at + n))
            total[o] += n
            at, left = at + n, left - n
    return chunks


def _pairs_of(case, ids):
    """The most-loaded device and the mask of the pairs it computes."""
    flat = ids.reshape(-1)
    loads = np.bincount(flat, minlength=case["E"])
    chunks = _plan_share(case, loads)
    rows = [0] * case["P"]
    for d, _, a, b in chunks:
        rows[d] += b - a
    top = rows.index(max(rows))
    on = np.zeros(flat.shape, dtype=bool)
    order = np.argsort(flat, kind="stable")
    first = np.concatenate([[0], np.cumsum(loads)])
    for d, e, a, b in chunks:
        if d == top:
            on[order[first[e] + a:first[e] + b]] = True
    return top, on


def _blocks(p, k):
    """Matrices p [E, n, k] in the packed order: blocks of 16 n x 32 k."""
    E, n, kk = p.shape
    return p.reshape(E, n // 16, 16, kk // 32, 32).transpose(2, 3).contiguous()


def exact(case, seed):
    s = _inputs(case, seed)
    E, D, F, T, K = (case[k] for k in ("E", "D", "F", "T", "K"))
    wg, wu, wd = s["w_gate"], s["w_up"], s["w_down"]
    if case["kind"] == "pack":
        # gate and up columns alternate in runs of 32
        both = torch.stack([wg.reshape(E, D, F // 32, 32), wu.reshape(E, D, F // 32, 32)], 3)
        both = both.reshape(E, D, 2 * F)
        gu = _blocks(both.transpose(1, 2), D).reshape(E, 2 * F, D)
        dn = _blocks(wd.transpose(1, 2), F).reshape(E, D, F)
        gut = _blocks(both, 2 * F).reshape(E, D, 2 * F)
        dnt = _blocks(wd, D).reshape(E, F, D)
        return gu, dn, gut, dnt
    ids = s["ids"].reshape(-1).long()
    on = torch.ones(T * K, dtype=torch.bool, device="cuda")
    if case["kind"] == "share":
        on = torch.from_numpy(_pairs_of(case, s["ids"].cpu().numpy())[1]).cuda()
    gates = s["gates"].reshape(-1).double()
    x, train = s["x"].double(), case["kind"] == "train"
    y = torch.zeros(T, D, dtype=torch.float64, device="cuda")
    if train:
        dy = s["dy"].double()
        dx, dgates = torch.zeros_like(y), torch.zeros_like(gates)
        dw = [torch.zeros(w.shape, dtype=torch.float64, device="cuda") for w in (wg, wu, wd)]
    for e in torch.unique(ids).tolist():
        p = torch.nonzero((ids == e) & on).reshape(-1)
        if p.numel() == 0:
            continue
        t = p // K
        a, b, c = wg[e].double(), wu[e].double(), wd[e].double()
        g, u = x[t] @ a, x[t] @ b
        sg = torch.sigmoid(g)
        act = g * sg * u
        out = act @ c
        y.index_add_(0, t, gates[p, None] * out)
        if train:
            dgates[p] = (dy[t] * out).sum(1)
            do = gates[p, None] * dy[t]
            da = do @ c.t()
            dg, du = da * u * sg * (1 + g * (1 - sg)), da * g * sg
            dx.index_add_(0, t, dg @ a.t() + du @ b.t())
            dw[0][e], dw[1][e], dw[2][e] = x[t].t() @ dg, x[t].t() @ du, act.t() @ do
    return (y, dx, dgates.reshape(T, K), *dw) if train else y
