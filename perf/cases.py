"""What a serving program has libsgmv do, as cases that can be timed and compared.

A case is one model invocation's worth of add-ons of one kind: the token rows of a batch, grouped into
segments by adapter, go through the same entry point once per layer, every layer with its own
activations, outputs and (stacked behind one pointer per adapter) weights.  That is how the paper's
runner uses the operator -- the segment indices are built once per invocation and serve all of its
layers -- and it keeps the weights coming from HBM rather than from the on-die caches.

Fields of a case
  call        "add_lora", "shrink", "expand", "multi" (projections that read the same activations in one
              call) or "layer" (all seven projections of a decoder layer through ``LoraLayer``)
  dtype       "f16" or "bf16"
  h_in, h_out widths of the projection; for "layer" the model width and the width of its MLP
  r           LoRA rank
  layers      layers of the invocation
  scale       LoRA's alpha / r
  proj        "multi": number of projections
  decode      token rows of requests in their decode phase, one each
  mix         how these requests share adapters: "distinct", "uniform", "skewed" or "identical"
  prompts     requests in their prefill phase, each with its own adapter and ...
  shortest, longest  ... a prompt of that many rows
  lengths     instead of the four fields above: the segment lengths themselves, "1,3,2,2"
  batch       seed of the batch's adapter ids and prompt lengths
  hint        whether the caller states the longest segment
  graph       whether the invocation is recorded once into a HIP graph and replayed
"""
from __future__ import annotations

import math
import random

import torch

from paper_2310_18547_amd import binding as B
from paper_2310_18547_amd.layer import GROUPS, PROJECTIONS, LoraLayer, projection_shapes

RANKS = (8, 16, 32, 64)
ADAPTERS = 64            # adapters the uniform and skewed mixes draw from
POOL_PAD = 64 * 1024     # adapters lie at a stride of their size plus this, as device.py and AdapterPool place them
TORCH = {"f16": torch.float16, "bf16": torch.bfloat16}
CODE = {"f16": B.F16, "bf16": B.BF16}

_DEFAULTS = dict(call="add_lora", dtype="f16", h_in=4096, h_out=4096, r=16, layers=32, scale=1.0, proj=1, decode=0,
                 mix="distinct", prompts=0, shortest=0, longest=0, lengths="", batch=0, hint=True, graph=False)


def _case(**fields):
    return {**_DEFAULTS, **fields}


def listed():
    return [
        # the smallest call: four requests of one to three rows on a 256-wide layer; launch and host cost
        _case(name="tiny", h_in=256, h_out=256, r=8, layers=1, lengths="1,3,2,2"),
        # one user: a single decode row of a Llama-7B-sized model, latency of 32 dependent calls
        _case(name="decode_1", decode=1),
        # the headline batch: 64 requests, each with its own adapter, the invocation recorded in a HIP graph
        _case(name="decode_distinct_64_graph", decode=64, graph=True),
        # a decode step of all seven projections, popular adapters shared by several requests
        _case(name="decode_layer_uniform_64", call="layer", h_out=11008, decode=64, mix="uniform", batch=3),
        # an odd batch with a few very popular adapters at the width of a 13B model, bfloat16
        _case(name="decode_skewed_45_bf16", h_in=5120, h_out=5120, r=32, layers=40, dtype="bf16", decode=45, mix="skewed",
              batch=5),
        # the widest decode projection at the highest rank: MLP down projection, every request its own adapter
        _case(name="decode_down_r64_bf16", h_in=13824, h_out=5120, r=64, layers=8, dtype="bf16", decode=64),
        # a large decode batch: the weights of 512 adapters per layer
        _case(name="decode_distinct_512", decode=512, layers=8),
        # the two steps on their own, for callers that put something between them (MLP-shaped, one per direction)
        _case(name="shrink_13824", call="shrink", h_in=13824, h_out=13824, decode=64, mix="uniform", batch=7),
        _case(name="expand_13824_r64_bf16", call="expand", h_in=13824, h_out=13824, r=64, dtype="bf16", decode=64, layers=16),
        # prompts of eight requests, square projection and MLP-sized output
        _case(name="prefill_8192_bf16", h_in=8192, h_out=8192, dtype="bf16", prompts=8, shortest=128, longest=1024, layers=4,
              batch=0),
        _case(name="prefill_mlp_r64_bf16", h_in=8192, h_out=28672, r=64, dtype="bf16", prompts=8, shortest=128, longest=1024,
              layers=2, batch=0),
        # the paper's running batch: a few prompts next to the decode rows of everybody else, q / k / v in one call
        _case(name="mixed_qkv", call="multi", proj=3, decode=41, mix="distinct", prompts=3, shortest=64, longest=512, layers=16,
              batch=11),
    ]


def _log_uniform(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def _width(rng):
    """Usual widths, and every other one: a multiple of 8 in [256, 13824]."""
    if rng.random() < 0.5:
        return rng.choice((1024, 2048, 4096, 5120, 8192, 11008, 13824))
    return max(256, _log_uniform(rng, 256, 13824) // 8 * 8)


def draw(rng):
    kind = rng.choice(("decode", "decode", "decode", "shrink", "expand", "multi", "layer", "prefill", "prefill_multi", "mixed"))
    c = _case(dtype=rng.choice(("f16", "bf16")), r=rng.choice(RANKS), h_in=_width(rng), h_out=_width(rng),
              scale=rng.choice((0.5, 1.0, 2.0)), batch=rng.randrange(1 << 20), hint=rng.random() < 0.9,
              graph=rng.random() < 0.2)
    mixes = ("distinct", "uniform", "skewed", "identical")
    if kind in ("decode", "shrink", "expand", "multi", "layer"):
        c.update(decode=_log_uniform(rng, 1, 512 if kind in ("decode", "shrink", "expand") else 128), mix=rng.choice(mixes))
    else:
        c.update(prompts=rng.randint(1, 8), shortest=_log_uniform(rng, 16, 128), longest=_log_uniform(rng, 128, 1024))
        if kind == "mixed":
            c.update(decode=_log_uniform(rng, 1, 128), mix=rng.choice(mixes))
            kind = rng.choice(("prefill", "prefill_multi"))
    if kind in ("shrink", "expand"):
        c["call"] = kind
    elif kind in ("multi", "prefill_multi"):
        c.update(call="multi", proj=rng.randint(2, 3))
    elif kind == "layer":
        c.update(call="layer", h_in=rng.choice((2048, 4096, 5120)))
        c["h_out"] = {2048: 5504, 4096: 11008, 5120: 13824}[c["h_in"]]
    # as many layers as the listed cases have, but no more than about 0.7 GB of traffic
    c["layers"] = 1
    c["layers"] = max(1, min(_log_uniform(rng, 1, 40), int(7e8 / work(c)["bytes"])))
    return c


def segments(case):
    """Segment lengths of the batch; every segment has an adapter of its own."""
    if case["lengths"]:
        return [int(n) for n in case["lengths"].split(",")]
    rng = random.Random(case["batch"])
    lens = [rng.randint(case["shortest"], case["longest"]) for _ in range(case["prompts"])]
    n, mix = case["decode"], case["mix"]
    if n and mix == "distinct":
        lens += [1] * n
    elif n and mix == "identical":
        lens.append(n)
    elif n:
        weights = [1.0 if mix == "uniform" else (i + 1.0) ** -1.5 for i in range(ADAPTERS)]  # Zipf(1.5): the paper's skewed mix
        count = {}
        for i in rng.choices(range(ADAPTERS), weights, k=n):
            count[i] = count.get(i, 0) + 1
        lens += [count[i] for i in sorted(count)]
    return lens


def _groups(case):
    """What one layer's calls read and write: (h_in, h_out, projections that share the input) of each call."""
    if case["call"] == "layer":
        shapes = projection_shapes(case["h_in"], case["h_out"])
        return [(*shapes[names[0]], len(names)) for names in GROUPS]
    return [(case["h_in"], case["h_out"], case["proj"])]


def work(case):
    lens = segments(case)
    rows, adapters, r = sum(lens), len(lens), case["r"]
    by = ops = 0
    for h_in, h_out, proj in _groups(case):
        if case["call"] != "expand":
            by += 2 * (rows * h_in + proj * adapters * h_in * r)
            ops += 2 * proj * rows * h_in * r
        if case["call"] != "shrink":
            by += 2 * proj * (2 * rows * h_out + adapters * r * h_out)
            ops += 2 * proj * rows * h_out * r
        if case["call"] in ("shrink", "expand"):  # v, fp32: accumulated into, or read
            by += 4 * rows * r * (2 if case["call"] == "shrink" else 1)
    return {"bytes": by * case["layers"], "flops": ops * case["layers"]}


def tolerance(case):
    if case["call"] == "shrink":
        return {"rel": 1e-5}  # fp32 sums of exact products
    # y is rounded once to 16 bits; the operands of the second product keep at least 16 bits
    return {"rel": 1e-3} if case["dtype"] == "f16" else {"rel": 8e-3}


def _random(gen, shape, dtype, std=1.0):
    t = torch.empty(shape, dtype=dtype, device="cuda:0").normal_(generator=gen)
    return t if std == 1.0 else t.mul_(std)


def _adapters(gen, n, shape, dtype, std):
    """``n`` weights in one allocation, each behind its own pointer: (keep-alive, device array of pointers)."""
    size = math.prod(shape)
    stride = (2 * size + POOL_PAD + 255) // 256 * 256
    pool = _random(gen, (n * stride // 2,), dtype, std)
    return pool, pool.data_ptr() + stride * torch.arange(n, dtype=torch.int64, device="cuda:0")


def prepare(case, seed):
    gen = torch.Generator("cuda:0").manual_seed(seed)
    dtype, r, layers, call = TORCH[case["dtype"]], case["r"], case["layers"], case["call"]
    lens = segments(case)
    rows, n = sum(lens), len(lens)
    starts = [0]
    for length in lens:
        starts.append(starts[-1] + length)
    longest = max(lens) if case["hint"] else 0
    s = {"case": case, "n_segs": n, "seg_starts": torch.tensor(starts, dtype=torch.int32, device="cuda:0"), "keep": []}

    def weights(h_in, h_out):
        a, a_ptrs = _adapters(gen, n, (layers, h_in, r), dtype, h_in ** -0.5)
        b, b_ptrs = _adapters(gen, n, (layers, r, h_out), dtype, r ** -0.5)
        s["keep"] += [a, b]
        return a_ptrs, b_ptrs

    if call == "layer":
        shapes = projection_shapes(case["h_in"], case["h_out"])
        ptrs = {name: weights(*shapes[name]) for name in PROJECTIONS}
        s["layer"] = LoraLayer(case["h_in"], case["h_out"], r, layers, rows, CODE[case["dtype"]],
                               {name: p[0] for name, p in ptrs.items()}, {name: p[1] for name, p in ptrs.items()},
                               s["seg_starts"], n, longest)
        # the projections of a group read the same activations
        s["x"] = [_random(gen, (layers, rows, shapes[names[0]][0]), dtype) for names in GROUPS]
        s["y"] = {name: _random(gen, (layers, rows, shapes[name][1]), dtype) for name in PROJECTIONS}
    else:
        h_in, h_out, proj = case["h_in"], case["h_out"], case["proj"]
        pairs = [weights(h_in, h_out) for _ in range(proj)]
        s["A"], s["B"] = [p[0] for p in pairs], [p[1] for p in pairs]
        if call != "expand":
            s["x"] = _random(gen, (layers, rows, h_in), dtype)
        if call in ("shrink", "expand"):
            s["v"] = _random(gen, (layers, rows, r), torch.float32)
        if call != "shrink":
            s["y"] = [_random(gen, (layers, rows, h_out), dtype) for _ in range(proj)]
        size = max(B.sgmv_workspace_bytes_multi(rows, r, proj), 256)
        s["workspace"] = torch.empty(size, dtype=torch.uint8, device="cuda:0")
        B.sgmv_workspace_init(s["workspace"], size)
        s["problem"] = B.make_problem(CODE[case["dtype"]], h_in, h_out, r, layers, rows, workspace=s["workspace"],
                                      workspace_bytes=size, max_seg_len=longest, workspace_ready=1)
    if case["graph"]:
        results = _results(s)
        before = [t.clone() for t in results]
        _invoke(s)  # kernels are loaded and their limits set before anything is recorded
        for t, b in zip(results, before):
            t.copy_(b)
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _invoke(s)
    return s


def _results(s):
    """What the calls accumulate into: v of the stand-alone shrink, else y."""
    if s["case"]["call"] == "shrink":
        return [s["v"]]
    return list(s["y"].values()) if isinstance(s["y"], dict) else s["y"]


def _invoke(s):
    """One model invocation: every layer's calls on the current stream."""
    c, seg_starts, n = s["case"], s["seg_starts"], s["n_segs"]
    call, scale = c["call"], c["scale"]
    stream = torch.cuda.current_stream().cuda_stream
    if call == "layer":
        layer, x, y = s["layer"], s["x"], s["y"]
        for i in range(c["layers"]):
            for g, names in enumerate(GROUPS):
                layer.add_lora_group(names, [y[name][i] for name in names], [x[g][i]] * len(names), i, scale, stream)
        return
    p, A, Bp = s["problem"], s["A"], s["B"]
    for i in range(c["layers"]):
        if call == "add_lora":
            B.sgmv_add_lora(p, s["y"][0][i], s["x"][i], A[0], Bp[0], seg_starts, n, i, scale, stream)
        elif call == "multi":
            B.sgmv_add_lora_multi(p, [y[i] for y in s["y"]], [s["x"][i]] * c["proj"], A, Bp, seg_starts, n, i, scale, stream)
        elif call == "shrink":
            B.sgmv_shrink(p, s["v"][i], s["x"][i], A[0], seg_starts, n, i, stream)
        else:
            B.sgmv_expand(p, s["y"][0][i], s["v"][i], Bp[0], seg_starts, n, i, scale, stream)


def run(state):
    if "graph" in state:
        state["graph"].replay()
    else:
        _invoke(state)
    return _results(state)
