"""What a user of the quantized linear has it do, as cases that can be timed and compared.

A case is a dict of plain values; `prepare` turns it and a seed into what a program holds before the
call (packed weights, activations, a captured graph), `run` makes one pass through the public calls.
Four kinds:

  block    the four linears of one decoder block (QKV, O, gate+up, down; sizes from synth.py), each with
           an input of its own, the way a serving step or a prompt runs them
  layer    one linear of any size: the calls on shapes that no tuning table lists
  convert  offline: fp16 weights -> packed layer -> canonical codes (quantize, then export)
  search   offline: channel salience of a layer over two gradient samples, and the choice of the
           8-bit channels over the layers of a model

`entry` says how a linear is called: "fp16" is linear_fp16 (fp16 in, fp16 out, buffers from torch's
allocator), "two_calls" is quantize_activations followed by mixed_linear (no scratch), "graph" is
linear_fp16_static with the caller's outputs, captured once in a graph and replayed.
"""
import math

import torch

import paper_2412_14590_amd as mx
from paper_2412_14590_amd import synth

MODELS = {"8b": synth.LLAMA3_8B, "70b": synth.LLAMA31_70B}
SIGMA = synth.SIGMA
# no case multiplies more than this many (activation, weight) pairs; the weights of one case have at
# most as many elements as the largest linear of the larger block
MOST_MACS = 8192 * sum(k * n for k, n in synth.LLAMA3_8B.values())
MOST_WEIGHTS = 8192 * 57344


def listed():
    return [
        # one sequence being generated: a token through a block, called from Python; where launches,
        # host work and the latency of small kernels count
        {"name": "token_8b", "kind": "block", "model": "8b", "M": 1, "entry": "fp16", "grouped": False, "share": 0.1},
        # the same served from a captured graph through the call that allocates nothing
        {"name": "token_8b_graph", "kind": "block", "model": "8b", "M": 1, "entry": "graph", "grouped": False, "share": 0.1},
        # a full decode batch on the larger block: the weight stream with 16 activation rows
        {"name": "batch16_70b", "kind": "block", "model": "70b", "M": 16, "entry": "fp16", "grouped": False, "share": 0.1},
        # a larger serving batch, between decode and prompt sizes
        {"name": "batch48_8b", "kind": "block", "model": "8b", "M": 48, "entry": "fp16", "grouped": False, "share": 0.1},
        # a short prompt
        {"name": "prompt256_8b", "kind": "block", "model": "8b", "M": 256, "entry": "fp16", "grouped": False, "share": 0.1},
        # the usual prompt (a chunk of chunked prefill)
        {"name": "prompt2048_8b", "kind": "block", "model": "8b", "M": 2048, "entry": "fp16", "grouped": False, "share": 0.1},
        # a long prompt, the largest listed work
        {"name": "prompt8192_8b", "kind": "block", "model": "8b", "M": 8192, "entry": "fp16", "grouped": False, "share": 0.1},
        # a prompt of a ragged length on the larger block
        {"name": "prompt777_70b", "kind": "block", "model": "70b", "M": 777, "entry": "fp16", "grouped": False, "share": 0.1},
        # the paper's own granularity: scales per group of 128 on both sides
        {"name": "groupwise1024_8b", "kind": "block", "model": "8b", "M": 1024, "entry": "fp16", "grouped": True, "share": 0.1},
        # a small odd layer, activations quantized by a call of their own, no scratch
        {"name": "ragged_layer", "kind": "layer", "K": 1920, "N": 3003, "M": 77, "entry": "two_calls", "grouped": False, "share": 0.2},
        # offline conversion of the largest linear of the smaller block
        {"name": "convert_gate_up", "kind": "convert", "K": 4096, "N": 28672, "grouped": False, "share": 0.1},
        # offline search for the 8-bit channels
        {"name": "search_gate_up", "kind": "search", "K": 4096, "N": 28672, "layers": 32, "share": 0.1},
    ]


def _spread(rng, lo, hi):
    """A whole number in [lo, hi], uniform over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["block", "block", "block", "layer", "layer", "layer", "convert", "search"])
    grouped = rng.random() < 0.25
    share = rng.choice([0.0, 0.05, 0.1, 0.1, 0.2, 0.5])
    if kind == "block":
        model = rng.choice(["8b", "8b", "70b"])
        entry = rng.choice(["fp16", "fp16", "fp16", "two_calls", "graph"])
        macs = sum(k * n for k, n in MODELS[model].values())
        most = MOST_MACS // macs
        if entry == "graph":                      # decode batches are what is served from a graph
            most = 64
        return {"kind": kind, "model": model, "M": _spread(rng, 1, most), "entry": entry, "grouped": grouped, "share": share}
    K = 128 * _spread(rng, 4, 224)
    N = _spread(rng, 64, min(57344, MOST_WEIGHTS // K))
    if kind == "layer":
        return {"kind": kind, "K": K, "N": N, "M": _spread(rng, 1, min(8192, MOST_MACS // (K * N))),
                "entry": rng.choice(["fp16", "two_calls"]), "grouped": grouped, "share": share}
    N = max(N, 1024)
    while N * K > MOST_WEIGHTS // 4:
        N //= 2
    if kind == "convert":
        return {"kind": kind, "K": K, "N": N, "grouped": grouped, "share": share}
    return {"kind": kind, "K": K, "N": N, "layers": 4 * rng.randint(1, 12), "share": rng.choice([0.05, 0.1, 0.2])}


# ---- inputs -------------------------------------------------------------------------------------

def _shapes(case):
    """[(K, N, sigma)] of the case's linears."""
    if case["kind"] == "block":
        return [(k, n, SIGMA[case["model"]]) for k, n in MODELS[case["model"]].values()]
    return [(case["K"], case["N"], SIGMA["8b"])]


def _n8(N, share):
    return synth.n8_for(N, share)


def _weights(N, K, sigma, gen):
    """N(0, sigma), one output channel in 64 four times as large (as synth.make_w, made on the GPU)."""
    W = torch.randn((N, K), generator=gen, device="cuda", dtype=torch.float16)
    W *= sigma
    rows = torch.randperm(N, generator=gen, device="cuda")[: max(1, N // 64)]
    W[rows] *= 4.0
    return W


def _activations(M, K, gen):
    """N(0, 1), one input channel in 100 twenty times as large (as synth.make_x)."""
    x = torch.randn((M, K), generator=gen, device="cuda", dtype=torch.float16)
    cols = torch.randperm(K, generator=gen, device="cuda")[: max(1, round(0.01 * K))]
    x[:, cols] *= 20.0
    return x


def _salient(W, n8):
    """The n8 channels with the widest range, ascending: which ones are 8-bit changes no kernel's work."""
    return torch.topk(W.abs().amax(dim=1), n8).indices.sort().values.to(torch.int32)


def _layer(K, N, sigma, share, grouped, gen):
    W = _weights(N, K, sigma, gen)
    return mx.quantize_weights(W, _salient(W, _n8(N, share)), 128 if grouped else None)


def _group(case):
    return 128 if case.get("grouped") else None


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind = case["kind"]
    if kind == "convert":
        W = _weights(case["N"], case["K"], SIGMA["8b"], gen)
        return {"case": case, "W": W, "sal": _salient(W, _n8(case["N"], case["share"]))}
    if kind == "search":
        N, K = case["N"], case["K"]
        W = _weights(N, K, SIGMA["8b"], gen)
        grads = [(torch.randn((N, K), generator=gen, device="cuda", dtype=torch.float16) * 0.05) for _ in range(2)]
        sizes = [n for _, n in synth.LLAMA3_8B.values()]
        saliences = [torch.exp(torch.randn(sizes[i % 4], generator=gen, device="cuda")) for i in range(case["layers"])]
        return {"case": case, "W": W, "grads": grads, "saliences": saliences,
                "T": int(case["share"] * sum(s.numel() for s in saliences))}
    linears = []
    for K, N, sigma in _shapes(case):
        layer = _layer(K, N, sigma, case["share"], case.get("grouped"), gen)
        linears.append((_activations(case["M"], K, gen), layer))
    state = {"case": case, "linears": linears}
    if case["entry"] == "graph":
        outs = [torch.empty((x.shape[0], layer.N), dtype=torch.float16, device="cuda") for x, layer in linears]

        def step():
            for (x, layer), y in zip(linears, outs):
                mx.linear_fp16_static(x, layer, y, _group(case))

        step()                                    # kernels are loaded before the capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        state.update(graph=graph, outs=outs)
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "convert":
        layer = mx.quantize_weights(state["W"], state["sal"], _group(case))
        codes = mx.unpack_weights(layer)
        return {"packed": [layer.w8, layer.w4, layer.s8, layer.s4, layer.z4, layer.perm], "codes": codes}
    if kind == "search":
        salience = None
        for i, grad in enumerate(state["grads"]):
            salience = mx.channel_salience(state["W"], grad, out=salience, weight=1.0 / len(state["grads"]), accumulate=i > 0)
        chosen = mx.select_salient(state["saliences"], state["T"])
        # the lists one after another, and how long each is
        return {"salience": salience, "chosen": torch.cat(chosen), "counts": [c.numel() for c in chosen]}
    if case["entry"] == "graph":
        state["graph"].replay()
        return state["outs"]
    if case["entry"] == "two_calls":
        return [mx.linear(x, layer, _group(case)) for x, layer in state["linears"]]
    return [mx.linear_fp16(x, layer, _group(case)) for x, layer in state["linears"]]


# ---- what a pass cannot do without ---------------------------------------------------------------

def _packed_bytes(K, N, n8, grouped):
    """4-bit rows: half a byte per weight, a 2-byte scale and half a byte of zero point per group; 8-bit
    rows: a byte per weight and a 2-byte scale per channel or per group; a 4-byte channel index per row."""
    ng = K // 128
    return (N - n8) * (K / 2 + 2.5 * ng) + n8 * (K + 2 * (ng if grouped else 1)) + 4 * N


def work(case):
    kind = case["kind"]
    if kind == "convert":
        K, N = case["K"], case["N"]
        n8, ng = _n8(N, case["share"]), K // 128
        packed = _packed_bytes(K, N, n8, case["grouped"])
        # canonical codes: a byte per weight, 2-byte scales, a byte per zero point
        codes = N * K + (N - n8) * 3 * ng + n8 * 2 * (ng if case["grouped"] else 1) + 4 * N
        return {"bytes": 2 * N * K + packed + codes + 4 * n8, "flops": 4 * N * K}
    if kind == "search":
        K, N = case["K"], case["N"]
        sizes = [n for _, n in synth.LLAMA3_8B.values()]
        total = sum(sizes[i % 4] for i in range(case["layers"]))
        return {"bytes": 2 * N * K + 2 * 2 * N * K + 4 * N + 4 * total + 4 * int(case["share"] * total), "flops": 2 * 6 * N * K}
    M = case["M"]
    nbytes = flops = 0
    for K, N, _ in _shapes(case):
        nbytes += _packed_bytes(K, N, _n8(N, case["share"]), case.get("grouped")) + 2 * M * K + 2 * M * N
        flops += 2 * M * N * K
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # codes, scales, zero points and channel lists are whole: the same bytes
    if case["kind"] == "convert":
        return "exact"
    # sums of K products in fp32: 8e-8 (largest 5e-7) from the same in 64 bits at K = 4096; the channel
    # lists are whole numbers, chosen on the same given values
    if case["kind"] == "search":
        return {"rel": 1e-6, "max": 1e-5}
    # fp32 sums of exact integers, rounded once to fp16: the generic kernel's order of the sums, and 64-bit
    # sums rounded to fp16, differ from the default path by at most 1.2e-5 (one result in 500 by a last
    # place, which is 2^-10 of the value at most)
    return {"rel": 5e-5, "max": 4e-3}
