"""The work that a program has this library do, as timed cases: a layer of one GPU's share (routing, then
the megakernel) from a handful of decode tokens to the full prefill batches of the five workloads, a stack of
layers in one launch, a layer on routing that the caller supplies, and the routing on its own.

A case is a dict of plain values: what it runs and the share's shape.  Every case goes through the public
entry points of ``binding`` the way bench.py and the tests do: the handle, the workspace and the packed
weights are the program's own and are made once (``prepare``); ``run`` is one pass.
"""
import math

import torch

from paper_2609_21483_amd import binding as B
from paper_2609_21483_amd.calibrate import load_calib
from paper_2609_21483_amd.workloads import MoeShape

KEYS = ("what", "ranks", "tokens", "hidden", "ffn", "experts", "top_k", "local", "shared", "zipf", "layers", "calib")


def _case(name, *values):
    return dict(name=name, **dict(zip(KEYS, values)))


def listed():
    return [
        # the smallest share of the workloads: launches and latency only
        _case("tiny_layer", "layer", 4, 16, 128, 256, 8, 2, 8, 0, 0.0, 1, ""),
        # decode steps: a few tokens from each rank, where the experts' weights are the traffic
        _case("decode_fine", "layer", 4, 8, 2048, 768, 128, 8, 32, 0, 1.2, 1, ""),
        _case("decode_mixtral", "layer", 4, 16, 4096, 14336, 8, 2, 2, 0, 0.0, 1, ""),
        # a decode batch of an odd number of tokens, with always-on shared experts
        _case("decode_shared", "layer", 4, 37, 2048, 1408, 64, 6, 16, 2, 0.0, 1, ""),
        # a short prefill of a ragged batch: row tiles mostly partly filled
        _case("ragged_fine", "layer", 4, 333, 2048, 768, 128, 8, 32, 0, 1.2, 1, ""),
        # the full batches of the workloads, with their measured tables
        _case("mixtral_layer", "layer", 4, 1024, 4096, 14336, 8, 2, 2, 0, 0.0, 1, "mixtral_ep4"),
        _case("fine_layer", "layer", 4, 2048, 2048, 768, 128, 8, 32, 0, 1.2, 1, "fine_zipf"),
        _case("shared_layer", "layer", 4, 4096, 2048, 1408, 64, 6, 16, 2, 0.0, 1, "shared_routed"),
        # a router of the caller's own: tables from supplied ids, every expert local
        _case("supplied_layer", "supplied", 2, 1500, 1024, 2816, 16, 4, 16, 0, 0.0, 1, ""),
        # routing alone, without a handle (serving loops, graph capture), over many experts
        _case("route_many_experts", "route", 1, 8192, 2048, 64, 256, 8, 32, 0, 0.5, 1, ""),
        # one layer of the large stack, routed and run by itself
        _case("large_layer", "layer", 4, 8192, 4096, 1536, 128, 8, 32, 0, 0.75, 1, "large_stack"),
        # the benchmark's step: eight layers routed on three streams, then run in one stacked launch
        _case("large_stack", "stack", 4, 8192, 4096, 1536, 128, 8, 32, 0, 1.5, 8, "large_stack"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        what = rng.choice(["layer", "layer", "layer", "layer", "supplied", "route", "stack"])
        ranks = rng.choice([1, 2, 4, 4, 8])
        tokens = log_int(1, 16384 // ranks)
        hidden = 64 * log_int(2, 64)
        ffn = 64 * log_int(2, 96)
        experts = log_int(4, 256)
        top_k = rng.randint(1, min(8, experts))
        local = max(1, min(64, experts // rng.choice([1, 2, 4, 4, 8])))
        shared = rng.choice([0, 0, 0, 1, 2])
        zipf = rng.choice([0.0, 0.0, 0.5, 1.2])
        layers = rng.randint(2, 4) if what == "stack" else 1
        if what == "route":
            local, shared, ffn, ranks, tokens = 1, 0, 64, 1, ranks * tokens
            if 16 * tokens * (experts + 1) + 2 * experts * hidden > 90 << 20:
                continue
        weights = 6 * hidden * ffn * (local + shared) * layers
        flops = 6 * hidden * ffn * layers * (ranks * tokens * top_k * local / experts + shared * tokens)
        rows = ranks * tokens * min(top_k, local) + shared * tokens + 256 * (local + shared + 1)
        if weights <= 3 << 30 and flops <= 8e12 and rows * hidden * 2 < 3 << 30:
            return dict(zip(KEYS, (what, ranks, tokens, hidden, ffn, experts, top_k, local, shared, zipf, layers, "")))


def _shape(c):
    return MoeShape("case", 0, c["ranks"], c["tokens"], c["hidden"], c["ffn"], c["experts"], c["top_k"], c["local"],
                    c["shared"])


def _inputs(c, seed):
    """Everything drawn: tokens N(0, 1), gates and expert weights N(0, 0.02^2), the Zipf log-prior (a stack
    draws each layer's exponent below c["zipf"]), and supplied routing where the caller routes."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(std, *shape):
        return torch.randn(*shape, device="cuda", generator=g, dtype=torch.float32).mul_(std).to(torch.bfloat16)

    T, H, F, E, k = c["ranks"] * c["tokens"], c["hidden"], c["ffn"], c["experts"], c["top_k"]
    x = normal(1.0, T, H)
    yield x
    for layer in range(c["layers"]):
        d = dict(wg=normal(0.02, H, E), bias=None)
        if c["zipf"]:
            s = c["zipf"] * (float(torch.rand((), device="cuda", generator=g)) if c["what"] == "stack" else 1.0)
            pi = torch.rand(E, device="cuda", generator=g).argsort().double()
            d["bias"] = (-s * torch.log(pi + 1.0)).float()
        if c["what"] == "supplied":
            d["idx"] = torch.rand(T, E, device="cuda", generator=g).topk(k, dim=1).indices.to(torch.int32).contiguous()
            w = torch.rand(T, k, device="cuda", generator=g) + 0.05
            d["w"] = (w / w.sum(1, keepdim=True)).contiguous()
        if c["what"] != "route":
            El, S = c["local"], c["shared"]
            d["experts"] = [normal(0.02, El, H, F), normal(0.02, El, H, F), normal(0.02, El, F, H)]
            d["shared"] = [normal(0.02, S, H, F), normal(0.02, S, H, F), normal(0.02, S, F, H)] if S else [None] * 3
        yield d


def prepare(case, seed):
    c = case
    T, H, k = c["ranks"] * c["tokens"], c["hidden"], c["top_k"]
    it = _inputs(c, seed)
    st = dict(case=c, x=next(it), layers=[], side=[])
    calib = load_calib(c["calib"], torch.cuda.get_device_properties(0).multi_processor_count) if c["calib"] else None
    for d in it:
        if c["what"] != "route":
            d["layer"] = B.MoeLayer(_shape(c), *d.pop("experts"), *d.pop("shared"), calib=calib)
            d["y"] = torch.empty(T, H, dtype=torch.bfloat16, device="cuda")
        if c["what"] != "supplied":
            d["idx"] = torch.empty(T, k, dtype=torch.int32, device="cuda")
            d["w"] = torch.empty(T, k, dtype=torch.float32, device="cuda")
        st["layers"].append(d)
    if c["what"] == "stack":
        st["side"] = [torch.cuda.Stream() for _ in range(min(3, c["layers"]))]
    return st


def run(state):
    c, x, L = state["case"], state["x"], state["layers"]
    d = L[0]
    if c["what"] == "route":
        B.moe_route_topk_static(x.shape[0], c["hidden"], c["experts"], c["top_k"], x, d["wg"], d["bias"], d["idx"], d["w"])
        return dict(idx=d["idx"], w=d["w"])
    if c["what"] == "supplied":
        B.moe_build_tables(d["layer"].h, d["idx"])
        d["layer"].forward(x, d["idx"], d["w"], d["y"])
        return dict(y=d["y"])
    if c["what"] == "layer":
        d["layer"].route(x, d["wg"], d["bias"], d["idx"], d["w"])
        d["layer"].forward(x, d["idx"], d["w"], d["y"])
        return dict(idx=d["idx"], w=d["w"], y=d["y"])
    # the layers' routings are independent: spread over the side streams, joined before the one launch
    main, side = torch.cuda.current_stream(), state["side"]
    fork = torch.cuda.Event()
    fork.record(main)
    for s in side:
        s.wait_event(fork)
    for i, d in enumerate(L):
        d["layer"].route(x, d["wg"], d["bias"], d["idx"], d["w"], stream=side[i % len(side)])
    for s in side:
        join = torch.cuda.Event()
        join.record(s)
        main.wait_event(join)
    B.moe_forward_stack([d["layer"].h for d in L], x, [d["idx"] for d in L], [d["w"] for d in L],
                        [d["layer"].packed for d in L], [d["y"] for d in L])
    return dict(idx=[d["idx"] for d in L], w=[d["w"] for d in L], y=[d["y"] for d in L])


def work(case):
    """Routing reads x and the gate once and writes ids and weights; a layer reads the weights of the experts
    that have a token (as many as uniform routing would touch) and writes y.  6 H F operations per row."""
    c = case
    T, H, F, E, k, n = c["ranks"] * c["tokens"], c["hidden"], c["ffn"], c["experts"], c["top_k"], c["layers"]
    nbytes, flops = 2.0 * T * H, 0.0
    if c["what"] != "supplied":
        nbytes += n * (2.0 * H * E + 8.0 * T * k)
        flops += n * 2.0 * T * E * H
    else:
        nbytes += 8.0 * T * k
    if c["what"] != "route":
        touched = c["local"] * (1.0 - (1.0 - k / E) ** T) + c["shared"]
        nbytes += n * (6.0 * H * F * touched + 2.0 * T * H)
        flops += n * 6.0 * H * F * (T * k * c["local"] / E + c["shared"] * c["tokens"])
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # ids are those of the defined logits, so they are the same everywhere
    if case["what"] == "route":
        # fp32 exponentials and one division: 6e-8 and 2.5e-7 from the 64-bit values
        return {"rel": 2.5e-7, "max": 1e-6, "differ": 0.0}
    # y is bf16, over bf16 h and expert outputs: sums in another order (fp32 torch products with the same
    # roundings, other split factors) differ by up to 4.4e-4, and by 0.025 at single values
    return {"rel": 1.8e-3, "max": 0.1, "differ": 0.0}


def _defined_logits(x, wg, bias):
    """The logits the routing is defined on: fp32, one accumulator per (token, expert), ascending hidden
    index (a product of two bf16 values is exact in fp32)."""
    xt, wf = x.t().float().contiguous(), wg.float()
    acc = torch.zeros(x.shape[0], wg.shape[1], device=x.device)
    for h in range(wf.shape[0]):
        acc.addcmul_(xt[h, :, None], wf[h, None, :])
    return acc if bias is None else acc + bias


def exact(case, seed):
    c = case
    it = _inputs(c, seed)
    x = next(it)
    T, k, Tr = x.shape[0], c["top_k"], c["tokens"]
    out = dict(idx=[], w=[], y=[])
    for d in it:
        if c["what"] == "supplied":
            idx, w = d["idx"].long(), d["w"].double()
        else:
            l, idx = torch.sort(_defined_logits(x, d["wg"], d["bias"]), dim=1, descending=True, stable=True)
            idx = idx[:, :k]
            w = torch.softmax(l[:, :k].double(), dim=1)
        out["idx"].append(None)
        out["w"].append(w)
        if c["what"] == "route":
            continue
        y = torch.zeros(T, c["hidden"], dtype=torch.float64, device="cuda")

        def ffn(rows, w1, w3, w2):
            v = x[rows].double()
            return (torch.nn.functional.silu(v @ w1.double()) * (v @ w3.double())) @ w2.double()

        for e in range(c["local"]):
            g, j = torch.nonzero(idx == e, as_tuple=True)
            if g.numel():
                y[g] += w[g, j, None] * ffn(g, *(t[e] for t in d["experts"]))
        for s in range(c["shared"]):
            y[:Tr] += ffn(slice(0, Tr), *(t[s] for t in d["shared"]))
        out["y"].append(y)
    if c["what"] == "stack":
        return out
    if c["what"] == "supplied":
        return dict(y=out["y"][0])
    return {key: v[0] for key, v in out.items() if v}
