"""The workloads whose speed this library is judged by: expert-layer inference, expert-layer training and routing
statistics, each through the public entry points of `paper_2603_06626_amd.binding`.

A case is a dict of plain values.  `listed()` names the representative ones, `draw()` picks further ones from the
same ranges, `prepare()` makes what a program holds before the call (inputs, weights, workspaces), `run()` is one pass.

kind = "infer"  the routing of one batch (cached ids and gates) becomes a plan, and `layers` expert layers run forward on it
kind = "train"  the same with a forward and a backward pass of every layer
kind = "stats"  per-sequence routing statistics, co-activation and expert folding over cached ids

Sizes: T tokens, d model width, f expert width, E experts, k experts per token.  The widths and expert counts of the
named configurations are those of `workloads.CONFIGS`; the ragged ones lie between them.  `gates` says whether the gate
weights are attached to the plan once ("plan") or handed to every layer call ("call"); `ids` is the dtype of the cached ids.
"""
import math

import numpy as np
import torch

from paper_2603_06626_amd import binding as gr
from paper_2603_06626_amd import workloads as wl

BF16 = torch.bfloat16
STREAM = 900     # sub-stream of the seeded generators, apart from those of the named configurations


def listed():
    return [
        # one new token of one sequence: the latency end of decoding; six experts of 64 per layer are touched
        dict(name="decode_1", kind="infer", T=1, d=2048, f=1408, E=64, k=6, routing="zipf", ids="uint8", gates="plan", layers=4),
        # a small decoding batch on the widest layer: nearly every token pulls in experts of its own
        dict(name="decode_16_wide", kind="infer", T=16, d=4096, f=1536, E=128, k=8, routing="uniform", ids="uint8", gates="plan", layers=2),
        # a full decoding batch on narrow experts: a few dozen rows per expert, one of them hot
        dict(name="decode_200", kind="infer", T=200, d=1024, f=512, E=64, k=8, routing="uniform_hot", ids="int32", gates="plan", layers=4),
        # a chunk of a prompt, widths and counts that are multiples of 8 and of nothing larger; gates come with the call
        dict(name="prefill_ragged", kind="infer", T=999, d=1928, f=1000, E=60, k=5, routing="zipf", ids="uint8", gates="call", layers=1),
        # forward pass of configuration 1 (narrow experts, uniform routing)
        dict(name="prefill_4096", kind="infer", T=4096, d=1024, f=512, E=64, k=8, routing="uniform", ids="int32", gates="plan", layers=1),
        # forward pass of configuration 2 (skewed routing: the hottest expert holds ten times the mean)
        dict(name="prefill_8192", kind="infer", T=8192, d=2048, f=1408, E=64, k=6, routing="zipf", ids="int32", gates="plan", layers=1),
        # training step of configuration 0: small enough that launches and latencies are what it costs
        dict(name="train_256", kind="train", T=256, d=128, f=256, E=8, k=2, routing="zipf", ids="int32", gates="plan", layers=1),
        # training micro-batch with ragged everything
        dict(name="train_ragged", kind="train", T=3001, d=1032, f=680, E=48, k=3, routing="zipf", ids="uint8", gates="call", layers=1),
        # training step of configuration 3, the benchmark's workload
        dict(name="train_8192", kind="train", T=8192, d=2048, f=1408, E=64, k=6, routing="zipf", ids="int32", gates="plan", layers=1),
        # one layer of configuration 4, the largest
        dict(name="train_16384", kind="train", T=16384, d=4096, f=1536, E=128, k=8, routing="uniform_hot", ids="int32", gates="plan", layers=1),
        # the statistics of a cached corpus shard (workloads.CORPUS)
        dict(name="stats_corpus", kind="stats", S=2048, L=4096, E=128, k=8, nodes=4, fold=32, ids="uint8", d=2048),
        # the same for the sequences of one batch, with int32 ids and a ragged length
        dict(name="stats_batch", kind="stats", S=48, L=1000, E=64, k=6, nodes=8, fold=10, ids="int32", d=1000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A multiple of 8, mostly one of 64 as real layers have, spread over the logarithm."""
    step = rng.choice((64, 64, 8))
    return max(step, (_log_int(rng, lo, hi) + step // 2) // step * step)


def draw(rng):
    """One more case of the same ranges, never dearer than the largest listed one."""
    while True:
        kind = rng.choice(("infer", "infer", "train", "train", "stats"))
        if kind == "stats":
            E = rng.choice((32, 60, 64, 128, 128, 200))
            c = dict(kind=kind, S=_log_int(rng, 32, 2048), L=_log_int(rng, 256, 4096), E=E, k=rng.randint(2, 8),
                     nodes=rng.choice((2, 4, 8, 16)), fold=rng.randint(E // 8, E // 2), ids=rng.choice(("uint8", "int32")),
                     d=_width(rng, 256, 4096))
        else:
            E = rng.choice((8, 16, 48, 64, 64, 96, 128))
            c = dict(kind=kind, T=_log_int(rng, 1, 16384) if kind == "infer" else _log_int(rng, 128, 16384),
                     d=_width(rng, 128, 4096), f=_width(rng, 256, 1536), E=E, k=rng.randint(1, min(8, E // 2)),
                     routing=rng.choice(("zipf", "uniform", "uniform_hot")), ids=rng.choice(("uint8", "int32")),
                     gates=rng.choice(("plan", "plan", "call")), layers=rng.randint(1, 4) if kind == "infer" else rng.randint(1, 2))
        w, most = work(c), work(next(x for x in listed() if x["name"] == "train_16384"))
        if w["flops"] <= most["flops"] and w["bytes"] <= most["bytes"]:
            return c


def _device():
    return torch.device("cuda:0")


def _prepare_stats(case, seed):
    dev = _device()
    S, L, E, k, n = case["S"], case["L"], case["E"], case["k"], case["nodes"]
    ids = wl.draw_sequence_routing(S, L, E, k, n_topics=4, seed=seed, stream=STREAM, device=dev, dtype=case["ids"])
    bits = np.zeros(E, dtype=np.uint64)
    for node, members in enumerate(wl.draw_expert_placement(E, n, seed=seed, stream=STREAM)):
        bits[members] |= np.uint64(1) << np.uint64(node)
    return dict(kind="stats", case=case, ids=ids, nodes=torch.from_numpy(bits.view(np.int64)).to(dev),
                score_w=torch.from_numpy(wl.draw_score_weights(case["d"], E, seed=seed, stream=STREAM)).to(dev),
                counts=torch.empty((S, E), dtype=torch.int32, device=dev), entropy=torch.empty(S, dtype=torch.float64, device=dev),
                loads=torch.empty(E, dtype=torch.int64, device=dev), maxvio=torch.empty(1, dtype=torch.float64, device=dev),
                comm=torch.empty((S, n), dtype=torch.int32, device=dev), best=torch.empty(S, dtype=torch.int32, device=dev),
                P=torch.empty((E, E), dtype=torch.int64, device=dev), group_of=torch.empty(E, dtype=torch.int32, device=dev),
                folded=torch.empty((case["d"], case["fold"]), dtype=torch.float32, device=dev))


def prepare(case, seed):
    if case["kind"] == "stats":
        return _prepare_stats(case, seed)
    dev = _device()
    T, d, f, E, k = case["T"], case["d"], case["f"], case["E"], case["k"]
    train = case["kind"] == "train"
    idx = wl.draw_routing(T, E, k, case["routing"], seed=seed, stream=STREAM, zipf_s=1.2)
    gates = torch.from_numpy(wl.draw_gates(T, k, seed=seed, stream=STREAM).view(np.int16)).to(dev).view(BF16)

    def normal(shape, sigma, tag, layer):
        return wl.draw_normal_bf16(shape, sigma, seed, STREAM, tag, layer, dev)

    layers = []
    for i in range(case["layers"]):
        layer = dict(x=normal((T, d), 1.0, "x", i), W1=normal((E, d, f), d ** -0.5, "W1", i), W3=normal((E, d, f), d ** -0.5, "W3", i),
                     W2=normal((E, f, d), f ** -0.5, "W2", i), y=torch.empty((T, d), dtype=BF16, device=dev))
        if train:
            layer.update(dY=normal((T, d), 1.0, "dY", i), dX=torch.empty((T, d), dtype=BF16, device=dev),
                         dW1=torch.empty((E, d, f), dtype=BF16, device=dev), dW3=torch.empty((E, d, f), dtype=BF16, device=dev),
                         dW2=torch.empty((E, f, d), dtype=BF16, device=dev),
                         ctx=torch.empty(gr.grouter_ctx_bytes(T, k, d, f), dtype=torch.uint8, device=dev))
        layers.append(layer)
    ws = gr.grouter_bwd_scratch_bytes(T, k, d, f) if train else gr.grouter_fwd_only_bytes(T, k, d, f)
    return dict(kind=case["kind"], case=case, ids=torch.from_numpy(idx).to(getattr(torch, case["ids"])).to(dev), gates=gates, layers=layers,
                plan=torch.empty(gr.grouter_plan_bytes(T, k, E), dtype=torch.uint8, device=dev),
                ws=torch.empty(ws, dtype=torch.uint8, device=dev))


def run(state):
    case = state["case"]
    if state["kind"] == "stats":
        E, flat = case["E"], state["ids"].view(-1, case["k"])
        gr.grouter_sample_stats(state["ids"], E, state["counts"], state["entropy"], state["loads"], state["maxvio"], state["nodes"],
                                case["nodes"], state["comm"], state["best"])
        gr.grouter_coactivation(flat, E, state["P"])
        gr.grouter_fold_groups(state["P"], case["fold"], state["group_of"])
        gr.grouter_fold_weights(state["score_w"], state["group_of"], case["fold"], state["folded"])
        return {n: state[n] for n in ("counts", "entropy", "loads", "maxvio", "comm", "best", "P", "group_of", "folded")}
    plan, k, ws = state["plan"], case["k"], state["ws"]
    gr.grouter_plan_build(state["ids"], case["E"], plan)
    gates = state["gates"]
    if case["gates"] == "plan":
        gr.grouter_plan_set_gates(plan, case["E"], gates)
        gates = None
    if state["kind"] == "infer":
        for s in state["layers"]:
            gr.grouter_moe_fwd_only(plan, s["x"], gates, s["W1"], s["W3"], s["W2"], s["y"], ws, k=k)
        return [s["y"] for s in state["layers"]]
    for s in state["layers"]:
        gr.grouter_moe_fwd(plan, s["x"], gates, s["W1"], s["W3"], s["W2"], s["y"], s["ctx"], k=k)
    for s in reversed(state["layers"]):
        gr.grouter_moe_bwd(plan, s["x"], gates, s["W1"], s["W3"], s["W2"], s["dY"], s["ctx"], s["dX"], s["dW1"], s["dW3"], s["dW2"], ws, k=k)
    return [[s[n] for n in ("y", "dX", "dW1", "dW3", "dW2")] for s in state["layers"]]


def _experts_touched(case):
    """Expected number of experts that at least one of T tokens picks (k distinct ones each, drawn without replacement)."""
    T, E, k = case["T"], case["E"], case["k"]
    p = [r ** -1.2 if case["routing"] == "zipf" else 1.0 for r in range(1, E + 1)]
    lo, hi = 0.0, 1e9
    for _ in range(200):     # inclusion probability 1 - exp(-z p) with the z that makes them add up to k
        z = 0.5 * (lo + hi)
        lo, hi = (z, hi) if sum(-math.expm1(-z * q) for q in p) < k else (lo, z)
    return sum(1.0 - math.exp(-z * q * T) for q in p)


def work(case):
    if case["kind"] == "stats":
        S, L, E, k = case["S"], case["L"], case["E"], case["k"]
        ids = S * L * k * (1 if case["ids"] == "uint8" else 4)
        out = S * E * 4 + S * 8 + E * 8 + 8 + S * case["nodes"] * 4 + S * 4 + E * E * 8 + E * 4 + case["d"] * case["fold"] * 4
        return {"bytes": ids + E * 8 + case["d"] * E * 4 + out, "flops": 0}
    T, d, f, E, k = case["T"], case["d"], case["f"], case["E"], case["k"]
    routing = T * k * ((1 if case["ids"] == "uint8" else 4) + 2)
    weights = 6 * d * f * _experts_touched(case)
    per_layer = weights + 4 * T * d                       # weights of the experts in use, x in, y out
    if case["kind"] == "train":
        per_layer += 4 * T * d + 6 * d * f * E            # dY in, dX out, weight gradients of every expert
    return {"bytes": routing + case["layers"] * per_layer,
            "flops": case["layers"] * (18 if case["kind"] == "train" else 6) * T * k * d * f}


def tolerance(case):
    if case["kind"] == "stats":
        # whole numbers are exact; entropies are fp64 sums, folded weights fp32 sums of at most E terms
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    # measured against the same formulas in fp64: 2-norm 2.9e-3 (forward) to 3.3e-3 (with gradients), largest element
    # 0.01 to 0.042 of max(rms, |value|); four times that
    return {"rel": 1.2e-2, "max": 0.16}
