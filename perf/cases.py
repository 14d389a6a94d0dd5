"""The workloads this library is timed on, through its public entry points.

A case is one call pattern of a user's program: a decode step (1 to 16 tokens,
fp16 activations), a prefill (a prompt's tokens, bf16 activations) or the
packing of a layer's weights at load time.  Shapes are those of the Llama2-13B
and Qwen3-32B layers the benchmark and the tests use, the single 2048 x 2048
linear, and generic ones; the bit mixes are the benchmark's 3, 4, 5 and 6 bit
budgets.

Fields of a case: ``op`` ("decode", "prefill", "pack"); ``net`` (which linears
one pass runs: "linear", "qkv", "mlp_in" = gate and up, "down", "layer" = the
layer's four launches); ``hidden`` (input channels of qkv and mlp_in, the
linear's k), ``q``, ``kv``, ``inter`` (output channels; the linear's n is
``q``); ``m`` tokens; ``bits`` average bits; ``clustered`` (the activations come
in clustered channel order, as a producer packed for its consumer emits them);
``scaled`` (per-channel factors are folded into the activations).
"""
import math

import numpy as np
import torch

import paper_2607_14618_amd as pq

DEV = "cuda"
GROUP = 128
QUANTUM = 32

# Percent of the channels at 2, 3, 4, 8 and 16 bits for each average budget.
MIXES = {3: (45, 35, 16, 3, 1), 4: (20, 30, 34.5, 14.5, 1), 5: (10, 20, 37, 32, 1), 6: (5, 10, 32, 52, 1)}
BITS = (2, 3, 4, 8, 16)


def _case(name, op, net, hidden, q, kv=0, inter=0, m=1, bits=3, clustered=False, scaled=False):
    return {"name": name, "op": op, "net": net, "hidden": hidden, "q": q, "kv": kv, "inter": inter, "m": m,
            "bits": bits, "clustered": clustered, "scaled": scaled}


def listed():
    return [
        # one small projection of one token: launch and latency bound
        _case("decode_2048_m1", "decode", "linear", 2048, 2048, m=1),
        # the attention input projections of one token
        _case("decode_qkv13b_m1", "decode", "qkv", 5120, 5120, kv=5120, m=1),
        # one token through all linears of a layer: the step a chat session repeats
        _case("decode_layer13b_m1", "decode", "layer", 5120, 5120, kv=5120, inter=13824, m=1),
        # the widest launch of a 32B layer at a larger budget, input emitted in its channel order
        _case("decode_mlp32b_m1_6b", "decode", "mlp_in", 5120, 8192, inter=25600, m=1, bits=6, clustered=True),
        # four concurrent sessions (or draft tokens), with activation-aware channel factors
        _case("decode_layer13b_m4", "decode", "layer", 5120, 5120, kv=5120, inter=13824, m=4, scaled=True),
        # the widest decode batch of one call, at 4 bits
        _case("decode_layer13b_m16", "decode", "layer", 5120, 5120, kv=5120, inter=13824, m=16, bits=4),
        # a ragged linear and a short prompt
        _case("prefill_ragged_m77", "prefill", "linear", 2976, 1357, m=77),
        # a short prompt (or a chunk of one) through a layer
        _case("prefill_layer13b_m33", "prefill", "layer", 5120, 5120, kv=5120, inter=13824, m=33, bits=4),
        # a prompt of 512 tokens: the grouped-query projections of a 32B layer, scaled
        _case("prefill_qkv32b_m512", "prefill", "qkv", 5120, 8192, kv=1024, m=512, bits=4, scaled=True),
        # a prompt of 512 tokens through all linears of a layer
        _case("prefill_layer13b_m512", "prefill", "layer", 5120, 5120, kv=5120, inter=13824, m=512, bits=4),
        # a long prompt: 2000 tokens of gate and up, input in clustered order
        _case("prefill_mlp13b_m2000", "prefill", "mlp_in", 5120, 5120, inter=13824, m=2000, bits=3, clustered=True),
        # loading: a quantized projection packed into the device layout
        _case("pack_13b_up", "pack", "linear", 5120, 13824, bits=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    top = max(_cost(c) for c in listed())
    while True:
        op = rng.choice(["decode"] * 5 + ["prefill"] * 5 + ["pack"])
        net = "linear" if op == "pack" else rng.choice(["linear", "linear", "qkv", "mlp_in", "down", "layer"])
        hidden = QUANTUM * _log_int(rng, 16, 400 if net != "linear" else 800)
        q = _log_int(rng, 128, 16000)
        kv = max(64, q // rng.choice([1, 1, 4, 8]))
        inter = QUANTUM * _log_int(rng, 32, 800)
        m = _log_int(rng, 1, 16) if op == "decode" else _log_int(rng, 17, 2048)
        c = _case("", op, net, hidden, q, kv, inter, m, rng.choice([3, 3, 4, 5, 6]), rng.random() < 0.3,
                  op != "pack" and rng.random() < 0.25)
        if net == "layer":
            c["q"] = QUANTUM * max(4, q // QUANTUM)  # the o projection reads q channels
        del c["name"]
        if _cost(c) <= top:
            return c


# --------------------------------------------------------------------------- inputs
def _launches(case):
    """(k, [n of each linear]) of each launch of one pass; a launch's linears share their input."""
    h, q, kv, inter = case["hidden"], case["q"], case["kv"], case["inter"]
    every = {"linear": [(h, [q])], "qkv": [(h, [q, kv, kv])], "mlp_in": [(h, [inter, inter])],
             "down": [(inter, [h])], "layer": [(h, [q, kv, kv]), (q, [h]), (h, [inter, inter]), (inter, [h])]}
    return every[case["net"]]


def _blocks(k, bits):
    """Channels of each bit-width, multiples of 32 that sum to k, nearest the mix (largest remainders)."""
    units = k // QUANTUM
    ideal = [p * units / 100 for p in MIXES[bits]]
    have = [int(v) for v in ideal]
    for i in sorted(range(len(ideal)), key=lambda i: have[i] - ideal[i])[: units - sum(have)]:
        have[i] += 1
    return [(b, u * QUANTUM) for b, u in zip(BITS, have) if u]


def _groups(blocks):
    return sum(-(-n // GROUP) for b, n in blocks if b < 16)


def _input(case, k, gen):
    """The activations of one launch, its permutation and its factors: N(0, 1) with 1 % of the channels
    50 times larger, those channels among the widest bit-widths, ascending channels inside a block."""
    blocks = _blocks(k, case["bits"])
    order = torch.randperm(k, generator=gen, device=DEV)
    x = torch.randn((case["m"], k), generator=gen, device=DEV)
    x[:, order[: max(1, k // 100)]] *= 50
    perm, at = [], 0
    for b, n in reversed(blocks):
        perm.insert(0, order[at: at + n].sort().values)
        at += n
    perm = torch.cat(perm).to(torch.int32)
    scale = None
    if case["scaled"]:
        scale = torch.exp2(torch.randint(-3, 4, (k,), generator=gen, device=DEV).float()).half()
    return blocks, perm, x.to(torch.float16 if case["op"] == "decode" else torch.bfloat16), scale


def _weights(n, k, blocks, gen):
    """Codes int16 [n][k] in clustered order, fp16 scales and zero points [n][groups]: N(0, 0.02^2)
    weights, asymmetric min-max per row and group of 128 channels of a block; 16 bits: the fp16 weight."""
    codes = torch.empty((n, k), dtype=torch.int16, device=DEV)
    scales, zeros, at = [], [], 0
    for b, length in blocks:
        w = torch.randn((n, length), generator=gen, device=DEV) * 0.02
        if b == 16:
            codes[:, at: at + length] = w.half().view(torch.int16)
        for lo, hi in ((0, length // GROUP * GROUP), (length // GROUP * GROUP, length)) if b < 16 else ():
            if lo == hi:
                continue
            g = w[:, lo:hi].view(n, -1, min(GROUP, hi - lo))
            low, high, top = g.amin(2, keepdim=True), g.amax(2, keepdim=True), (1 << b) - 1
            s = ((high - low) / top).half()
            z = torch.clamp(torch.round(-low / s.float()), 0, top)
            c = torch.clamp(torch.round(g / s.float()) + z, 0, top)
            codes[:, at + lo: at + hi] = c.view(n, hi - lo).to(torch.int16)
            scales.append(s.squeeze(2))
            zeros.append(z.half().squeeze(2))
        at += length
    return codes, torch.cat(scales, 1), torch.cat(zeros, 1)


def _inputs(case, seed):
    """Every launch of the case: (blocks, perm, x, factors, [weights of each linear]), one at a time."""
    for i, (k, ns) in enumerate(_launches(case)):
        gen = torch.Generator(device=DEV)
        gen.manual_seed(1000003 * int(seed) + i)
        blocks, perm, x, scale = _input(case, k, gen)
        yield blocks, perm, x, scale, (_weights(n, k, blocks, gen) for n in ns)


def prepare(case, seed):
    """Packed weights, permutations, activations and the launches' handles (pack: the quantized weights)."""
    state = {"op": case["op"], "launches": []}
    for blocks, perm, x, scale, weights in _inputs(case, seed):
        if case["op"] == "pack":
            codes, scales, zeros = next(weights)
            return {"op": "pack", "layout": pq.plan(*codes.shape, blocks), "weights": (codes, scales, zeros)}
        given = pq.permute(perm, x) if case["clustered"] else x
        items = []
        for codes, scales, zeros in weights:
            layout = pq.plan(*codes.shape, blocks)
            items.append((layout, pq.pack(layout, codes, scales, zeros), None if case["clustered"] else perm, given,
                          None, scale))
        state["launches"].append(pq.PreparedBatch("gemv" if case["op"] == "decode" else "gemm", items))
    return state


def run(state):
    if state["op"] == "pack":
        return pq.pack(state["layout"], *state["weights"])
    return [launch.run() for launch in state["launches"]]


# --------------------------------------------------------------------------- what a pass costs and gives
def work(case):
    nbytes = flops = 0
    for k, ns in _launches(case):
        blocks = _blocks(k, case["bits"])
        code_bits = sum(b * n for b, n in blocks)
        for n in ns:
            packed = n * code_bits // 8 + 4 * n * _groups(blocks)
            if case["op"] == "pack":
                return {"bytes": packed + 2 * n * k + 4 * n * _groups(blocks), "flops": 0}
            nbytes += packed + 4 * case["m"] * n
            flops += 2 * case["m"] * n * k
        nbytes += 2 * case["m"] * k + (0 if case["clustered"] else 4 * k) + (2 * k if case["scaled"] else 0)
    return {"bytes": nbytes, "flops": flops}


def _cost(case):
    """Seconds of a pass at the card's nominal rates, about."""
    w = work(case)
    return w["bytes"] / 4e12 + w["flops"] / 6e14


def tolerance(case):
    # bytes of the packed layout; or fp32 sums of exact products: 0.6e-7 to 1.1e-7 from the 64-bit
    # result over these cases, and as far again for the longest input
    return "exact" if case["op"] == "pack" else {"rel": 6e-7}


def exact(case, seed):
    if case["op"] == "pack":
        return None
    out = []
    for blocks, perm, x, scale, weights in _inputs(case, seed):
        xc = x.double().index_select(1, perm.long())
        if scale is not None:
            xc = xc * scale.double()
        ys = []
        for codes, scales, zeros in weights:
            w = torch.empty(codes.shape, dtype=torch.float64, device=DEV)
            at = g = 0
            for b, length in blocks:
                part = codes[:, at: at + length]
                if b == 16:
                    w[:, at: at + length] = part.contiguous().view(torch.float16).double()
                else:
                    groups = -(-length // GROUP)
                    of = torch.arange(length, device=DEV) // GROUP + g
                    w[:, at: at + length] = scales.double()[:, of] * (part.double() - zeros.double()[:, of])
                    g += groups
                at += length
            ys.append(xc @ w.T)
        out.append(ys)
    return [[np.asarray(y.cpu()) for y in ys] for ys in out]
