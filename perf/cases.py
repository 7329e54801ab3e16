"""Performance cases of the resident-expert MoE layer: what a program that serves with this framework asks of it.

A pass is one layer forward on a batch of token rows that is already in HBM, through the public entry points and into
buffers that the program keeps (`LayerBuffers`, allocated once per layer and batch shape).  Inputs follow the recipe of
`emoe_inputs`: x ~ N(0, 1), weights ~ N(0, 1/fan_in), a Zipf-distributed gate bias where a layer has popular experts, a
part of the experts resident, and no token whose choice of experts hangs on the last bits of its gate logits.
"""
from __future__ import annotations

import math

import torch

import paper_2503_06823_amd as P

DEVICE = "cuda:0"


def _case(name, T, d, f, E, k, R, S=0, dtype="bf16", act="swiglu", zipf=0.0, resident="seeded", calls="one"):
    """T tokens, d_model d, d_ff f, E experts of which R are resident in S slots, k experts per token.  `calls`: "one" =
    emoe_layer_forward; "four" = route, permute, expert FFN and combine called one by one (what a program does that
    looks at the routing in between); "observe" = the same four with the workload counted by the route call."""
    return {"name": name, "T": T, "d": d, "f": f, "E": E, "k": k, "R": R, "S": S or R, "dtype": dtype, "act": act,
            "zipf": zipf, "resident": resident, "calls": calls}


def listed():
    return [
        # the smallest call: the fp32 verification layer, a handful of launches on next to no data
        _case("tiny_f32", 64, 128, 256, 8, 2, 4, dtype="f32"),
        # fp32 at a working size: a Switch-style layer run in full precision (reference runs, numerics checks)
        _case("switch_1024_f32", 1024, 768, 3072, 64, 1, 16, dtype="f32", act="relu", zipf=1.1),
        # a Switch-style layer, top-1 of 64 experts, ReLU: small weights, launch-bound
        _case("switch_1024", 1024, 768, 3072, 64, 1, 16, act="relu", zipf=1.1),
        # one user's decode step at the Mixtral-8x7B shape: one token, two experts' weights
        _case("decode_1", 1, 4096, 14336, 8, 2, 6),
        # a batch of 64 users' decode step at that shape, 6 of 8 experts resident
        _case("decode_64", 64, 4096, 14336, 8, 2, 6),
        # a decode batch of 128 with every expert resident: around 32 rows per expert
        _case("decode_128", 128, 4096, 14336, 8, 2, 8),
        # one short prompt at that shape
        _case("prompt_256", 256, 4096, 14336, 8, 2, 6),
        # two prompts of 512 tokens with every expert resident (the first prompts of a run)
        _case("prompts_1024", 1024, 4096, 14336, 8, 2, 8),
        # the prefill of a batch of eight prompts, half the experts resident: the headline layer
        _case("prefill_4096", 4096, 4096, 14336, 8, 2, 4),
        # a fine-grained layer: 64 small experts, six per token, the 24 most popular resident
        _case("finegrained_8192", 8192, 2048, 1408, 64, 6, 24, zipf=1.2, resident="popular"),
        # an OpenMoE-shaped layer with popular experts (slots from a few rows to most of the batch), in a program that
        # observes the experts' workload to choose the next resident set
        _case("openmoe_2048_observed", 2048, 2048, 8192, 32, 2, 16, zipf=1.1, calls="observe"),
        # nothing is a multiple of a tile: odd token count, extents of 8 modulo 64, empty slots, top-3
        _case("ragged_357", 357, 1032, 2808, 24, 3, 11, S=20, zipf=1.1, calls="four"),
    ]


def _mats(c):
    return 3 if c["act"] == "swiglu" else 2


def _elem(c):
    return 4 if c["dtype"] == "f32" else 2


def _flops(c):
    return 2.0 * c["T"] * c["k"] * _mats(c) * c["d"] * c["f"] + 2.0 * c["T"] * c["d"] * c["E"]


def _weight_bytes(c):
    return c["R"] * _mats(c) * c["d"] * c["f"] * _elem(c)


# bounds of the drawn cases: no more matrix work than the prefill layer, no more weights than eight Mixtral experts
_MOST_FLOPS = 2.9e12
_MOST_WEIGHT_BYTES = 8 * 3 * 4096 * 14336 * 2
_MOST_F32_FLOPS = 1.5e10
_MOST_F32_WEIGHT_BYTES = 512 << 20


def draw(rng):
    """One more layer of the ranges above: 1 to 8192 tokens, d_model 128 to 6144, d_ff 256 to 16384, 4 to 64 experts,
    top-1 to top-8, a quarter to all of them resident; fp32 layers up to the size of the listed one."""
    def log_uniform(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    def extent(lo, hi, grain):
        return max(lo, int(round(log_uniform(lo, hi) / grain)) * grain)

    while True:
        dtype = "f32" if rng.random() < 0.125 else "bf16"
        grain = 128 if rng.random() < 0.5 else 8
        d, f = extent(128, 1024 if dtype == "f32" else 6144, grain), extent(256, 4096 if dtype == "f32" else 16384, grain)
        E = int(round(log_uniform(4, 64)))
        k = min(int(round(log_uniform(1, 8))), E)
        R = rng.randint(max(k, (E + 3) // 4), E)
        S = min(E, R + (rng.randint(1, 4) if rng.random() < 0.25 else 0))
        T = int(round(log_uniform(1, 8192)))
        c = _case("", T, d, f, E, k, R, S, dtype, "relu" if rng.random() < 0.25 else "swiglu",
                  rng.choice((0.0, 0.0, 1.1, 1.2)), rng.choice(("seeded", "popular")), rng.choice(("one", "one", "four", "observe")))
        del c["name"]
        f32 = dtype == "f32"
        if (_flops(c) <= (_MOST_F32_FLOPS if f32 else _MOST_FLOPS)
                and _weight_bytes(c) <= (_MOST_F32_WEIGHT_BYTES if f32 else _MOST_WEIGHT_BYTES)
                and T * k * max(d, f) <= 1 << 28):
            return c


MARGIN = 1e-4  # smallest gap between the gate logits that decide a token's experts


def _close_rows(logits, k):
    """Rows whose k + 1 largest logits have two closer together than MARGIN."""
    top = logits.topk(min(k + 1, logits.shape[1]), dim=1).values
    return (top[:, :-1] - top[:, 1:] < MARGIN).any(dim=1).nonzero().flatten()


def prepare(case, seed):
    """A layer's weights in their slots, its slot map, a batch of token rows and the layer's buffers, all on the GPU."""
    c = dict(case)
    dtype = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))

    def normal(shape, std):
        return torch.empty(shape, dtype=dtype, device=DEVICE).normal_(0.0, std, generator=g)

    T, d, f, E, k, R, S = (c[n] for n in ("T", "d", "f", "E", "k", "R", "S"))
    rank = torch.randperm(E, generator=g, device=DEVICE)
    bias = -c["zipf"] * torch.log(1.0 + rank.float()) if c["zipf"] > 0 else None
    experts = rank.argsort()[:R] if c["resident"] == "popular" else torch.randperm(E, generator=g, device=DEVICE)[:R]
    slots = torch.randperm(S, generator=g, device=DEVICE)[:R]
    slot_of_expert = torch.full((E,), -1, dtype=torch.int32, device=DEVICE)
    slot_of_expert[experts] = slots.to(torch.int32)

    w_gate = normal((E, d), d ** -0.5)
    x = normal((T, d), 1.0)
    rows = torch.arange(T, device=DEVICE)
    while rows.numel():  # the few rows that are too close to call are drawn again
        logits = x[rows].double() @ w_gate.double().t()
        if bias is not None:
            logits += bias.double()
        close = [_close_rows(logits[:, slot_of_expert >= 0], k)]
        if c["calls"] == "observe":
            close.append(_close_rows(logits, k))
        rows = rows[torch.cat(close).unique()]
        if rows.numel():
            x[rows] = normal((rows.numel(), d), 1.0)

    desc = P.make_desc(T, d, f, E, k, S, c["dtype"], c["act"])
    return {"calls": c["calls"], "buf": P.LayerBuffers.allocate(desc, DEVICE),
            "layer": (w_gate, bias, slot_of_expert, normal((S, f, d), d ** -0.5),
                      normal((S, f, d), d ** -0.5) if c["act"] == "swiglu" else None, normal((S, d, f), f ** -0.5)),
            "x": x, "expert_tokens": torch.zeros(E, dtype=torch.int64, device=DEVICE)}


def run(state):
    """One forward of the layer; the layer's output, the routing and the slots' row counts."""
    b, x, layer = state["buf"], state["x"], state["layer"]
    outputs = {"out": b.out, "topk_expert": b.topk_expert, "topk_weight": b.topk_weight, "slot_counts": b.slot_counts}
    if state["calls"] != "observe":
        P.layer_forward(b, x, *layer, one_call=state["calls"] == "one")
        return outputs
    w_gate, bias, slot_of_expert, w1, w3, w2 = layer
    d = b.desc
    P.emoe_route_observe(d, x, w_gate, bias, slot_of_expert, b.topk_expert, b.topk_weight, state["expert_tokens"])
    P.emoe_permute(d, x, b.topk_expert, slot_of_expert, b.slot_counts, b.slot_offsets, b.perm, b.inv_perm, None,
                   b.permute_ws, b.permute_ws.numel())
    P.emoe_expert_ffn_gather_combine(d, x, b.perm, b.inv_perm, b.slot_offsets, w1, w3, w2, b.topk_weight, b.y_perm,
                                     b.out, b.ffn_ws, b.ffn_ws.numel())
    outputs["expert_tokens"] = state["expert_tokens"]
    return outputs


def work(case):
    """Token rows in, output rows out, the gate and the weights of the slots that receive rows once each; the routed
    rows' matrix work.  The slots in use are the expected number under the layer's popularity."""
    c = case
    weight = [1.0] * c["R"]
    if c["zipf"] > 0:  # share of a resident expert by rank; residents spread over the ranks unless they are the popular ones
        step = 1.0 if c["resident"] == "popular" else c["E"] / c["R"]
        weight = [(1.0 + i * step) ** -c["zipf"] for i in range(c["R"])]
    total = sum(weight)
    used = sum(1.0 - (1.0 - min(1.0, c["k"] * w / total)) ** c["T"] for w in weight)
    el = _elem(c)
    return {"bytes": 2 * c["T"] * c["d"] * el + c["E"] * c["d"] * el + used * _mats(c) * c["d"] * c["f"] * el,
            "flops": _flops(c)}


def tolerance(case):
    """About four times what the layer's output differs from the same layer computed in 64 bits: bf16 2.9e-3 (largest
    0.016), where h and y are each rounded once to 8 bits; fp32 8.6e-7 (largest 5.2e-6), where only sums are rounded."""
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 2e-5}
    return {"rel": 1e-2, "max": 7e-2}
