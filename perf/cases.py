"""Timed workloads of the qwZ / qgZ path: what a training or serving program
has this package do, through its public entry points.

Sizes are those of the package's own workloads (`workloads.py`): a 1024 x 1024
tensor, one GPT-1.3B layer (hidden 2048), one GPT-20B layer (hidden 6144), and
the 123,456,789-element tensor that no block, word or slice count divides.
`draw` spreads over the same ranges.  A case's "op" says which calls it makes:

  path     a small tensor through all five calls: quantise and dequantise the
           weight, quantise the gradient, reduce, dequantise
  weights  the forward side: quantise this rank's shard into its slot of the
           gathered buffer, dequantise the gathered layer
  encode   one quantiser call over a whole tensor (INT8 weight or INT4 gradient)
  levels   the backward side: reduce levels of the given fan-ins, one after the
           other, then the gradient shard's dequantisation
  fused    a last level fused with the dequantisation
  gather   a level whose slices lie in separate buffers (addresses in host
           arrays, or in device tables that the program keeps)
  layer    the four weight products of a GPT layer at some number of tokens
           (QKV 3h x h, attention output h x h, FC1 4h x h, FC2 h x 4h), the
           weights held as gathered INT8
  gemm     one such product

Inputs are drawn on the GPU with plain torch: weights N(0, 0.02), gradients
N(0, 1e-3), activations N(0, 1), and for the stress tensor Student-t values
with outliers and all-zero groups.
"""
import math

import torch

import paper_2501_04266_amd as zq

DEV = "cuda"
N_TINY = 1024 * 1024
N_13B = 12 * 2048 * 2048
N_20B = 12 * 6144 * 6144
N_EDGE = 123_456_789
_DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_SIZE = {"f32": 4, "f16": 2, "bf16": 2}


def listed():
    return [
        # the smallest: every call of the path on 1M elements or fewer, bound by
        # launches and by the calls' own cost
        {"name": "tiny-path", "op": "path", "n": N_TINY, "dtype": "f16", "wblock": 256, "gblock": 128, "P": 2},
        # forward of a GPT-20B layer sharded 8 ways: bf16 weights, INT8 blocks of 256
        {"name": "20b-weights", "op": "weights", "n": N_20B, "shard": 8, "block": 256, "dtype": "bf16",
         "out": "bf16"},
        # backward of the same layer: the whole fp32 gradient to INT4 blocks of 128
        {"name": "20b-grad-encode", "op": "encode", "bits": 4, "n": N_20B, "block": 128, "dtype": "f32",
         "values": "grad"},
        # its three-level reduce-scatter (GCD pair, node, 48 nodes) and the shard for the optimizer
        {"name": "20b-3level", "op": "levels", "m": N_20B // 2, "fanins": "2,4,48", "block": 128, "out": "f32"},
        # a GPT-1.3B layer's one-level reduce-scatter over 8 ranks, fused with the dequantisation
        {"name": "1.3b-fused-p8", "op": "fused", "m": N_13B // 8, "P": 8, "block": 128, "out": "f32"},
        # the same level with each peer's slice read where it lies, without allocation
        {"name": "1.3b-gather-p8", "op": "gather", "m": N_13B // 8, "P": 8, "block": 128, "tables": False},
        # the stress tensor: ragged length, outliers and zero groups, fp32 to INT8
        {"name": "edge-encode", "op": "encode", "bits": 8, "n": N_EDGE, "block": 256, "dtype": "f32",
         "values": "outlier"},
        # the ragged tensor's gradient reduced over 8 ranks: an odd shard (15,432,099 elements), so
        # slices start at odd byte addresses; the shard dequantised to bf16
        {"name": "edge-level-p8", "op": "levels", "m": -(-N_EDGE // 8), "fanins": "8", "block": 64, "out": "bf16"},
        # decode: 16 tokens through a GPT-20B layer whose weights stay INT8
        {"name": "20b-layer-16", "op": "layer", "h": 6144, "M": 16, "block": 256, "dtype": "bf16"},
        # a small batch, fp16 activations
        {"name": "20b-layer-64", "op": "layer", "h": 6144, "M": 64, "block": 256, "dtype": "f16"},
        # a prefill of a few hundred tokens
        {"name": "20b-layer-512", "op": "layer", "h": 6144, "M": 512, "block": 256, "dtype": "bf16"},
        # the largest: FC1 at a training micro-batch of 8192 tokens
        {"name": "20b-fc1-8192", "op": "gemm", "M": 8192, "N": 24576, "K": 6144, "block": 256, "dtype": "bf16"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["path", "weights", "encode", "levels", "fused", "gather", "layer", "gemm", "gemm"])
    block = rng.choice([64, 128, 128, 256, 256, 512])
    if op == "path":
        P = rng.choice([2, 4, 8])
        n = _log(rng, 1 << 16, 1 << 23) // P * P
        return {"op": op, "n": n, "dtype": rng.choice(["f16", "bf16", "f32"]), "wblock": rng.choice([128, 256]),
                "gblock": rng.choice([64, 128]), "P": P}
    if op == "weights":
        shard = rng.choice([1, 2, 8])
        # a shard's slot of the gathered buffer starts at a whole block
        n = max(1, _log(rng, 1 << 18, N_20B) // (shard * block)) * shard * block
        if shard == 1:
            n += rng.randrange(block)
        return {"op": op, "n": n, "shard": shard, "block": block, "dtype": rng.choice(["f16", "bf16", "f32"]),
                "out": rng.choice(["bf16", "f16", "f32"])}
    if op == "encode":
        bits = rng.choice([4, 8])
        return {"op": op, "bits": bits, "n": _log(rng, 1 << 18, N_20B // 2), "block": block,
                "dtype": rng.choice(["f32", "f32", "bf16", "f16"]), "values": rng.choice(["grad", "outlier"])}
    if op in ("levels", "fused", "gather"):
        P = rng.choice([2, 3, 4, 6, 8, 8, 12, 16, 32, 48, 64])
        m = max(1, _log(rng, 1 << 20, N_20B // 2) // P)
        if rng.random() < 0.6:  # shards are usually padded to whole blocks
            m = max(1, m // block) * block
        case = {"op": op, "m": m, "block": block}
        if op == "levels":
            case.update(fanins=str(P), out=rng.choice(["f32", "bf16"]))
        elif op == "fused":
            case.update(P=P, out=rng.choice(["f32", "bf16"]))
        else:
            case.update(P=P, tables=rng.random() < 0.5)
        return case
    dtype = rng.choice(["bf16", "bf16", "f16"])
    if op == "layer":
        return {"op": op, "h": rng.choice([2048, 6144]), "M": _log(rng, 1, 1024), "block": rng.choice([128, 256]),
                "dtype": dtype}
    h = rng.choice([2048, 4096, 6144])
    N, K = rng.choice([(3 * h, h), (h, h), (4 * h, h), (h, 4 * h)])
    if rng.random() < 0.25:  # an output width that no tile divides
        N -= rng.randrange(1, 64)
    return {"op": op, "M": _log(rng, 1, 8192), "N": N, "K": K, "block": rng.choice([128, 256]), "dtype": dtype}


# ---------------------------------------------------------------- inputs (plain torch)

def _randn(n, std, gen, dtype="f32"):
    return (torch.randn(n, generator=gen, device=DEV) * std).to(_DT[dtype])


def _values(n, values, gen, dtype):
    if values == "weight":
        return _randn(n, 0.02, gen, dtype)
    if values == "grad":
        return _randn(n, 1e-3, gen, dtype)
    # Student-t with 3 degrees of freedom, one element in a thousand 100 times
    # larger, one aligned group of 256 in a hundred zero
    x = torch.randn(n, generator=gen, device=DEV)
    x *= 0.02
    chi = torch.zeros(n, device=DEV)
    for _ in range(3):
        chi += torch.randn(n, generator=gen, device=DEV).square_()
    x *= chi.div_(3.0).rsqrt_()
    del chi
    x[torch.randint(0, n, (n // 1000,), generator=gen, device=DEV)] *= 100.0
    groups = n // 256
    if groups:
        at = torch.randint(0, groups, (groups // 100 + 1,), generator=gen, device=DEV)
        x[: groups * 256].view(groups, 256)[at] = 0.0
    return x.to(_DT[dtype])


def _blocks(x, block):
    """x as rows of one block each, the last one padded with zeros."""
    short = -x.numel() % block
    return (torch.nn.functional.pad(x, (0, short)) if short else x).view(-1, block)


def _encode(x, block, qmax):
    """Symmetric absmax codes (int8, one an element) and scales, in x's type."""
    b = _blocks(x, block)
    a = b.abs().amax(1)
    codes = torch.round(b * torch.where(a > 0, qmax / a, torch.zeros_like(a))[:, None]).to(torch.int8)
    return codes.view(-1)[: x.numel()], a / qmax


def _pack(codes):
    """Two codes a byte, the first in the low half."""
    if codes.numel() % 2:
        codes = torch.nn.functional.pad(codes, (0, 1))
    pair = codes.view(torch.uint8).view(-1, 2)
    return (pair[:, 0] & 15) | (pair[:, 1] << 4)


def _unpack(packed, m):
    low = (packed << 4).view(torch.int8) >> 4
    high = packed.view(torch.int8) >> 4
    return torch.stack((low, high), 1).view(-1)[:m]


def _slices(P, m, block, gen):
    """P INT4 slices of m gradient values each, as the peers send them."""
    packed, scales = [], []
    for _ in range(P):
        c, s = _encode(_randn(m, 1e-3, gen), block, 7.0)
        packed.append(_pack(c))
        scales.append(s)
    return packed, scales


def _fanins(case):
    """(P, m) of each level: a level's output is shared out over the next one's ranks."""
    m, got = case["m"], []
    for i, P in enumerate(int(p) for p in case["fanins"].split(",")):
        m = m if i == 0 else m // P
        got.append((P, m))
    return got


def _products(case):
    """(M, N, K) of the products of a layer or gemm case."""
    if case["op"] == "gemm":
        return [(case["M"], case["N"], case["K"])]
    M, h = case["M"], case["h"]
    return [(M, 3 * h, h), (M, h, h), (M, 4 * h, h), (M, h, 4 * h)]


def _inputs(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    op = case["op"]
    if op == "path":
        m = case["n"] // case["P"]
        packed, scales = _slices(case["P"], m, case["gblock"], gen)
        return {"w": _values(case["n"], "weight", gen, case["dtype"]), "g": _values(case["n"], "grad", gen, "f32"),
                "packed": torch.cat(packed), "scales": torch.cat(scales)}
    if op == "weights":
        codes, scales = _encode(_randn(case["n"], 0.02, gen), case["block"], 127.0)
        mine = case["n"] // case["shard"] if case["shard"] > 1 else case["n"]
        return {"codes": codes, "scales": scales, "w": _values(mine, "weight", gen, case["dtype"])}
    if op == "encode":
        return {"x": _values(case["n"], case["values"], gen, case["dtype"])}
    if op == "levels":
        got = [_slices(P, m, case["block"], gen) for P, m in _fanins(case)]
        return {"levels": [(torch.cat(p), torch.cat(s)) for p, s in got]}
    if op in ("fused", "gather"):
        packed, scales = _slices(case["P"], case["m"], case["block"], gen)
        if op == "fused":
            return {"packed": torch.cat(packed), "scales": torch.cat(scales)}
        return {"packed": packed, "scales": scales}
    products = []
    for M, N, K in _products(case):
        x = torch.randn(M * K, generator=gen, device=DEV).to(_DT[case["dtype"]]).view(M, K)
        codes, scales = _encode(_randn(N * K, 0.02, gen), case["block"], 127.0)
        products.append((x, codes, scales, N))
    return {"products": products}


# ---------------------------------------------------------------- the calls

def prepare(case, seed):
    state = _inputs(case, seed)
    state["case"] = case
    if case["op"] == "gather":
        # the level's output buffers, and the address tables where the program keeps them
        m, block = case["m"], case["block"]
        state["out"] = (torch.empty((m + 1) // 2, dtype=torch.uint8, device=DEV),
                        torch.empty(-(-m // block), dtype=torch.float32, device=DEV))
        if case["tables"]:
            state["tables"] = zq.gather_tables(state["packed"], state["scales"])
    return state


def run(state):
    case = state["case"]
    op = case["op"]
    if op == "path":
        m = case["n"] // case["P"]
        codes, scales = zq.qwz_quantize(state["w"], case["wblock"])
        w = zq.qwz_dequantize(codes, scales, case["wblock"], out_dtype=_DT[case["dtype"]])
        sent, sent_scales = zq.qgz_quantize(state["g"], case["gblock"])
        got, got_scales = zq.qgz_reduce_level(state["packed"], state["scales"], case["P"], m, case["gblock"])
        g = zq.qgz_dequantize(got, got_scales, m, case["gblock"])
        return codes, scales, w, sent, sent_scales, got, got_scales, g
    if op == "weights":
        block, n = case["block"], state["w"].numel()
        codes, scales = zq.qwz_quantize(state["w"], block, codes=state["codes"][:n],
                                        scales=state["scales"][: -(-n // block)])
        return codes, scales, zq.qwz_dequantize(state["codes"], state["scales"], block, out_dtype=_DT[case["out"]])
    if op == "encode":
        return (zq.qwz_quantize if case["bits"] == 8 else zq.qgz_quantize)(state["x"], case["block"])
    if op == "levels":
        outs = []
        for (P, m), (packed, scales) in zip(_fanins(case), state["levels"]):
            outs.append(zq.qgz_reduce_level(packed, scales, P, m, case["block"]))
        outs.append(zq.qgz_dequantize(*outs[-1], m, case["block"], out_dtype=_DT[case["out"]]))
        return outs
    if op == "fused":
        return zq.qgz_reduce_dequantize(state["packed"], state["scales"], case["P"], case["m"], case["block"],
                                        out_dtype=_DT[case["out"]])
    if op == "gather":
        packed, scales = state["out"]
        if case["tables"]:
            return zq.qgz_reduce_level_gather(state["packed"], state["scales"], case["m"], case["block"], packed,
                                              scales, tables=state["tables"])
        return zq.qgz_reduce_level_gather_noalloc(state["packed"], state["scales"], case["m"], case["block"], packed,
                                                  scales)
    return [zq.qwz_dequant_gemm(x, codes, scales, N, case["block"]) for x, codes, scales, N in state["products"]]


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    op, flops = case["op"], 0.0
    if op == "path":
        n, m = case["n"], case["n"] // case["P"]
        e, ws, gs = _SIZE[case["dtype"]], 4.0 / case["wblock"], 4.0 / case["gblock"]
        size = n * (2 * e + 2 + 2 * ws) + n * (4 + 0.5 + gs) + (case["P"] + 1) * m * (0.5 + gs) + m * (4.5 + gs)
        flops = 4.0 * n + 3.0 * n + 2.0 * case["P"] * m + 4.0 * m
    elif op == "weights":
        n, mine = case["n"], case["n"] // case["shard"]
        size = mine * (_SIZE[case["dtype"]] + 1 + 4.0 / case["block"]) + n * (
            1 + 4.0 / case["block"] + _SIZE[case["out"]])
        flops = 3.0 * mine + n
    elif op == "encode":
        size = case["n"] * (_SIZE[case["dtype"]] + case["bits"] / 8.0 + 4.0 / case["block"])
        flops = 3.0 * case["n"]
    elif op == "levels":
        one, size = 0.5 + 4.0 / case["block"], 0.0
        for P, m in _fanins(case):
            size += (P + 1) * m * one
            flops += 2.0 * P * m + 3.0 * m
        size += m * (one + _SIZE[case["out"]])
        flops += m
    elif op in ("fused", "gather"):
        one, P, m = 0.5 + 4.0 / case["block"], case["P"], case["m"]
        size = P * m * one + m * (_SIZE[case["out"]] if op == "fused" else one)
        flops = 2.0 * P * m + 3.0 * m
    else:
        size = 0.0
        for M, N, K in _products(case):
            size += 2.0 * M * K + N * K * (1 + 4.0 / case["block"]) + 4.0 * M * N
            flops += 2.0 * M * N * K
    return {"bytes": float(size), "flops": float(flops)}


def tolerance(case):
    # the codecs and the reduce levels are defined bit for bit
    if case["op"] not in ("layer", "gemm"):
        return "exact"
    # products are exact in binary32 and summed there: sums in another order
    # are this far apart
    return {"rel": 2e-6, "max": 2e-5}


# ---------------------------------------------------------------- in 64 bits

def _decode64(codes, scales, block):
    return (_blocks(codes.double(), block) * scales.double()[:, None]).view(-1)[: codes.numel()]


def _encode64(x, block, qmax):
    codes, scales = _encode(x.double(), block, qmax)
    return codes, scales


def _level64(packed, scales, P, m, block):
    """One level in 64 bits: the codes and scales of the requantised sum."""
    nbytes, nscales = (m + 1) // 2, -(-m // block)
    total = torch.zeros(m, dtype=torch.float64, device=DEV)
    for p in range(P):
        total += _decode64(_unpack(packed[p * nbytes:(p + 1) * nbytes], m), scales[p * nscales:(p + 1) * nscales],
                           block)
    return _encode64(total, block, 7.0)


def exact(case, seed):
    """None stands for codes: whole numbers, compared as such."""
    i, op = _inputs(case, seed), case["op"]
    if op == "path":
        m = case["n"] // case["P"]
        c, s = _encode64(i["w"], case["wblock"], 127.0)
        _, gs = _encode64(i["g"], case["gblock"], 7.0)
        rc, rs = _level64(i["packed"], i["scales"], case["P"], m, case["gblock"])
        return (None, s, _decode64(c, s, case["wblock"]), None, gs, None, rs, _decode64(rc, rs, case["gblock"]))
    if op == "weights":
        c, s = _encode64(i["w"], case["block"], 127.0)
        i["codes"][: c.numel()] = c
        scales = i["scales"].double()
        scales[: s.numel()] = s
        return None, s, _decode64(i["codes"], scales, case["block"])
    if op == "encode":
        return None, _encode64(i["x"], case["block"], 127.0 if case["bits"] == 8 else 7.0)[1]
    if op == "levels":
        outs = []
        for (P, m), (packed, scales) in zip(_fanins(case), i["levels"]):
            c, s = _level64(packed, scales, P, m, case["block"])
            outs.append((None, s))
        return outs + [_decode64(c, s, case["block"])]
    if op == "fused":
        return _decode64(*_level64(i["packed"], i["scales"], case["P"], case["m"], case["block"]), case["block"])
    if op == "gather":
        return None, _level64(torch.cat(i["packed"]), torch.cat(i["scales"]), case["P"], case["m"], case["block"])[1]
    outs = []
    for x, codes, scales, N in i["products"]:
        # the weight as the dequantiser defines it: fl32(code * scale), rounded to x's type
        w = (_blocks(codes.float(), case["block"]) * scales[:, None]).view(-1)[: codes.numel()]
        w = w.to(x.dtype).double().view(N, x.shape[1])
        outs.append(x.double() @ w.t().contiguous())
        del w
    return outs
