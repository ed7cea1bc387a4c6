"""The work this package does for its users, as a list of cases that can be timed and compared.

`listed()` gives the standing cases, `draw(rng)` one more of the same ranges.  `prepare` makes what a
program holds before the call (inputs from a seed, compressed weights, kept buffers), `run` is one
pass through the public entry points and returns its outputs, `work` the bytes and operations such a
pass cannot do without, `tolerance` how far two correct implementations may differ.

Kinds of case:
  layer    one linear layer: vnm_spmm, or vnm_spmm_fused where it has a bias or channel permutations
  block    the linear layers of one Transformer block, one call each, layers that read the same
           activations reading the same tensor.  family "llama": q, k, v, o, gate, up, down;
           family "deit": qkv, proj, fc1, fc2 with biases or without.  mode "call" uses vnm_spmm /
           vnm_spmm_fused, "bound" the functions vnm_spmm_bind gives to a decode loop, "shared"
           vnm_stage_x once per activation and vnm_spmm_staged per layer
  prune    vnm_prune_compress of a dense weight, and vnm_decompress back to the dense masked weight
  refresh  vnm_refresh_mask: merge of the LoRA matrices, RIA scores, pruning from the scores
  search   vnm_permutation_search on a score matrix
"""

from __future__ import annotations

import math

import torch

import paper_2410_16135_amd as vnm

DEV = "cuda:0"


def _layer(name, out, inn, tokens, V, M, fp32=False, bias=False, perm_in=False, perm_out=False):
    return {"name": name, "kind": "layer", "out": out, "in": inn, "tokens": tokens, "V": V, "M": M, "fp32": fp32,
            "bias": bias, "perm_in": perm_in, "perm_out": perm_out}


def _block(name, family, width, ffn, tokens, V, M, mode, bias=False):
    return {"name": name, "kind": "block", "family": family, "width": width, "ffn": ffn, "tokens": tokens, "V": V,
            "M": M, "mode": mode, "bias": bias}


def listed():
    return [
        # the smallest layer of the benchmark's configurations: latency and launches
        _layer("layer_128x128_t16", 128, 128, 16, 64, 8),
        # decoding one sequence with a Llama-2-7B block, its calls bound once as a serving loop does
        _block("llama_decode_t1", "llama", 4096, 11008, 1, 64, 5, "bound"),
        # decoding a batch of 24 sequences at a sparser pattern
        _block("llama_decode_t24", "llama", 4096, 11008, 24, 64, 8, "bound"),
        # a short prompt of a length that is no multiple of any tile
        _block("llama_prefill_t700", "llama", 4096, 11008, 700, 64, 5, "call"),
        # the benchmark's own workload: prefill of 4096 tokens, staging shared by q/k/v and by gate/up
        _block("llama_prefill_t4096", "llama", 4096, 11008, 4096, 64, 5, "shared"),
        # encoders: 64 images of 197 tokens through DeiT-small (with the layers' biases) and DeiT-base
        _block("deit_small_t12608", "deit", 384, 1536, 12608, 64, 5, "call", bias=True),
        _block("deit_base_t12608", "deit", 768, 3072, 12608, 64, 8, "call"),
        # a layer with its bias and both channel permutations merged in, 32-row blocks
        _layer("permuted_4096_t2048", 4096, 4096, 2048, 32, 8, bias=True, perm_in=True, perm_out=True),
        # a classifier-like layer of odd sizes in 16-row blocks, fp32 result
        _layer("odd_1000x1030_t333", 1000, 1030, 333, 16, 7, fp32=True),
        # preparing a layer, and the dense weight back for checking it
        {"name": "prune_11008x4096", "kind": "prune", "out": 11008, "in": 4096, "V": 64, "M": 5, "mask": False},
        # mask update of LoRA training with dynamic masks
        {"name": "refresh_4096x4096_r16", "kind": "refresh", "out": 4096, "in": 4096, "V": 64, "M": 5, "rank": 16},
        # channel permutations before pruning, two alternations
        {"name": "search_2048x2048", "kind": "search", "out": 2048, "in": 2048, "V": 64, "M": 5, "iterations": 2},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _width(rng, lo, hi, odd):
    """A layer width: a multiple of 8 as a rule, any number with probability `odd`."""
    n = _log_int(rng, lo, hi)
    return n if rng.random() < odd else max(8, (n + 4) // 8 * 8)


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "block", "block", "prune", "refresh", "search"])
    V, M = rng.choice([32, 64, 64, 128]), rng.choice([4, 5, 5, 6, 7, 8, 8, 10, 12, 16])
    if kind == "layer":
        out, inn = _width(rng, 96, 11008, 0.2), _width(rng, 96, 11008, 0.15)
        if rng.random() < 0.1:
            V = 16
        plain = V == 16 or inn % 8 != 0             # no matrix-core copy or no aligned rows
        cap = 4.0e9 if plain else 1.5e11            # tokens x out x in
        tokens = _log_int(rng, 1, int(max(1, min(12608, cap / (out * inn)))))
        fused = rng.random() < 0.3
        return _layer("", out, inn, tokens, V, M, fp32=rng.random() < 0.25, bias=fused,
                      perm_in=fused and rng.random() < 0.5, perm_out=fused and rng.random() < 0.5)
    if kind == "block":
        if rng.random() < 0.6:
            width = _width(rng, 512, 4096, 0.0)
            ffn = min(11008, (int(width * rng.uniform(2.5, 2.75)) + 7) // 8 * 8)
            tokens = _log_int(rng, 1, 4096)
            mode = "bound" if tokens <= 64 else rng.choice(["call", "shared"])
            return _block("", "llama", width, ffn, tokens, V, M, mode)
        width = _width(rng, 192, 768, 0.0)
        return _block("", "deit", width, 4 * width, _log_int(rng, 197, 12608), V, M, "call", bias=rng.random() < 0.5)
    if kind == "prune":
        return {"kind": "prune", "out": _width(rng, 96, 11008, 0.2), "in": _width(rng, 96, 11008, 0.15), "V": V, "M": M,
                "mask": rng.random() < 0.3}
    if kind == "refresh":
        return {"kind": "refresh", "out": _width(rng, 96, 4096, 0.2), "in": _width(rng, 96, 4096, 0.15), "V": V, "M": M,
                "rank": rng.choice([4, 8, 16, 16, 32])}
    return {"kind": "search", "out": _width(rng, 256, 2048, 0.3), "in": _width(rng, 256, 2048, 0.3), "V": rng.choice([32, 64]),
            "M": rng.choice([4, 5, 8]), "iterations": rng.choice([1, 2])}


def _layers(case):
    """(name, out, in, index of the activation tensor it reads) of a block's layers."""
    w, f = case["width"], case["ffn"]
    if case["family"] == "llama":
        return [("q", w, w, 0), ("k", w, w, 0), ("v", w, w, 0), ("o", w, w, 1), ("gate", f, w, 2), ("up", f, w, 2),
                ("down", w, f, 3)]
    return [("qkv", 3 * w, w, 0), ("proj", w, w, 1), ("fc1", f, w, 2), ("fc2", w, f, 3)]


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _weight(g, out, inn):
    """N(0, 0.02^2) with 1 % of the input columns ten times larger, in fp16."""
    W = torch.randn((out, inn), generator=g, device=DEV) * 0.02
    cols = torch.randperm(inn, generator=g, device=DEV)[: int(round(0.01 * inn))]
    W[:, cols] *= 10.0
    return W.to(torch.float16)


def _activations(g, tokens, inn):
    return torch.randn((tokens, inn), generator=g, device=DEV).to(torch.float16)


def prepare(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    st = {"case": case}
    if kind == "layer":
        st["c"] = vnm.vnm_prune_compress(_weight(g, case["out"], case["in"]), case["V"], case["M"])
        st["x"] = _activations(g, case["tokens"], case["in"])
        st["bias"] = torch.randn(case["out"], generator=g, device=DEV).to(torch.float16) if case["bias"] else None
        for p, n in (("perm_in", case["in"]), ("perm_out", case["out"])):
            st[p] = torch.randperm(n, generator=g, device=DEV).to(torch.int32) if case[p] else None
    elif kind == "block":
        T, M = case["tokens"], case["M"]
        layers = _layers(case)
        st["c"] = [vnm.vnm_prune_compress(_weight(g, o, i), case["V"], M) for _, o, i, _ in layers]
        widths = {x: i for _, _, i, x in layers}
        st["x"] = [_activations(g, T, widths[k]) for k in range(len(widths))]
        st["bias"] = [torch.randn(o, generator=g, device=DEV).to(torch.float16) if case["bias"] else None
                      for _, o, _, _ in layers]
        if case["mode"] == "bound":
            ws = torch.empty(max([vnm.vnm_spmm_workspace_bytes(T, c) for c in st["c"]] + [256]), dtype=torch.uint8,
                             device=DEV)
            st["calls"] = [vnm.vnm_spmm_bind(st["x"][x], c, torch.empty((T, o), dtype=torch.float16, device=DEV), ws)
                           for (_, o, _, x), c in zip(layers, st["c"])]
        elif case["mode"] == "shared":
            st["staged"] = [vnm.vnm_stage_x(x, M) for x in st["x"]]     # kept and overwritten by every pass
    elif kind == "prune":
        st["w"] = _weight(g, case["out"], case["in"])
    elif kind == "refresh":
        out, inn, r = case["out"], case["in"], case["rank"]
        st["w"] = _weight(g, out, inn)
        st["b"] = torch.randn((out, r), generator=g, device=DEV) * 0.01
        st["a"] = torch.randn((r, inn), generator=g, device=DEV) * 0.05
        st["act"] = torch.rand(inn, generator=g, device=DEV) * 2.0 + 0.1
    else:
        W = _weight(g, case["out"], case["in"])
        st["s"] = vnm.vnm_ria_scores(W, torch.rand(case["in"], generator=g, device=DEV) * 2.0 + 0.1)
        st["scale"] = float(2.0 ** 30 / float(st["s"].max()))
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "layer":
        dt = torch.float32 if case["fp32"] else torch.float16
        if case["bias"] or case["perm_in"] or case["perm_out"]:
            return vnm.vnm_spmm_fused(state["x"], state["c"], bias=state["bias"], perm_in=state["perm_in"],
                                      perm_out=state["perm_out"], out_dtype=dt)
        return vnm.vnm_spmm(state["x"], state["c"], out_dtype=dt)
    if kind == "block":
        if case["mode"] == "bound":
            return [call() for call in state["calls"]]
        layers = _layers(case)
        if case["mode"] == "shared":
            outs, done = [], -1
            for (_, _, _, x), c in zip(layers, state["c"]):
                if x != done:
                    vnm.vnm_stage_x(state["x"][x], case["M"], staged=state["staged"][x])
                    done = x
                outs.append(vnm.vnm_spmm_staged(state["staged"][x], case["tokens"], c))
            return outs
        if case["bias"]:
            return [vnm.vnm_spmm_fused(state["x"][x], c, bias=b)
                    for (_, _, _, x), c, b in zip(layers, state["c"], state["bias"])]
        return [vnm.vnm_spmm(state["x"][x], c) for (_, _, _, x), c in zip(layers, state["c"])]
    if kind == "prune":
        c = vnm.vnm_prune_compress(state["w"], case["V"], case["M"], want_mask=case["mask"])
        dense = vnm.vnm_decompress(c)
        # (the matrix-core copy is opaque and partly unwritten padding; the layer cases multiply by it)
        return [c.values, c.meta, c.colidx, dense] + ([c.mask] if case["mask"] else [])
    if kind == "refresh":
        c = vnm.vnm_refresh_mask(state["w"], state["b"], state["a"], 2.0, case["V"], case["M"], act=state["act"])
        return [c.values, c.meta, c.colidx, c.mask]
    perm_out, perm_in, history = vnm.vnm_permutation_search(state["s"], case["V"], case["M"], state["scale"],
                                                            iterations=case["iterations"])
    return [perm_out, perm_in, history]


def _triple_bytes(out, inn, V, M):
    s = vnm.vnm_query_sizes(out, inn, V, M)
    return 2 * s.values_elems + s.meta_bytes + s.colidx_bytes


def _packed_bytes(out, inn, V, M):
    return vnm.vnm_query_sizes(out, inn, V, M).packed_bytes


def _kept(out, inn, M):
    return 2 * out * -(-inn // M)


def work(case):
    kind, V, M = case["kind"], case["V"], case["M"]
    if kind == "layer":
        out, inn, T = case["out"], case["in"], case["tokens"]
        b = 2 * T * inn + (4 if case["fp32"] else 2) * T * out + _triple_bytes(out, inn, V, M)
        b += 2 * out * case["bias"] + 4 * inn * case["perm_in"] + 4 * out * case["perm_out"]
        return {"bytes": b, "flops": 2 * T * _kept(out, inn, M)}
    if kind == "block":
        T, layers = case["tokens"], _layers(case)
        b = sum(2 * T * i for i in {x: i for _, _, i, x in layers}.values())
        b += sum(2 * T * o + _triple_bytes(o, i, V, M) + 2 * o * case["bias"] for _, o, i, _ in layers)
        return {"bytes": b, "flops": sum(2 * T * _kept(o, i, M) for _, o, i, _ in layers)}
    out, inn = case["out"], case["in"]
    outputs = _triple_bytes(out, inn, V, M) + _packed_bytes(out, inn, V, M)
    if kind == "prune":     # W in; triple, matrix-core copy and dense W' out; a sum and a comparison per weight
        return {"bytes": 4 * out * inn + outputs + out * inn * case["mask"], "flops": 2 * out * inn}
    if kind == "refresh":   # W, B, A in; triple, matrix-core copy and mask out
        r = case["rank"]
        return {"bytes": 3 * out * inn + 4 * r * (out + inn) + 4 * inn + outputs, "flops": (2 * r + 6) * out * inn}
    # search: a maximum and a sum per row for every (lifted channel, block) of every round
    B, R = inn // M, -(-out // V)
    rounds = M * B * B * out + V * R * R * inn
    return {"bytes": 4 * out * inn + 4 * (out + inn), "flops": 2 * case["iterations"] * rounds}


def tolerance(case):
    """Pruning, merging and the search are defined to the bit.  A product accumulates in fp32 and is
    rounded once to its output type: against the same product in fp64 the relative 2-norm error is
    2.1e-4 with an fp16 result and, with an fp32 one, 1.1e-7 to 1.4e-6 from the shortest to the longest
    sums of these ranges; about four times that is stated."""
    if case["kind"] in ("prune", "refresh", "search"):
        return "exact"
    return {"rel": 5e-6 if case.get("fp32") else 8e-4}


def _masked64(W, V, M):
    """V:N:M pruning of W in fp64: per V x M block the four columns of largest L1 norm, per row the two
    largest magnitudes among them, ties to the lower index."""
    out, inn = W.shape
    R, B = -(-out // V), -(-inn // M)
    P = torch.zeros((R * V, B * M), dtype=torch.float64, device=W.device)
    P[:out, :inn] = W.double()
    P = P.reshape(R, V, B, M)
    norms = P.abs().sum(1)                                                          # [R, B, M], exact
    cols = torch.sort(norms, dim=-1, descending=True, stable=True).indices[..., :4].sort(-1).values
    cols = cols[:, None].expand(R, V, B, 4)
    kept = P.gather(3, cols)
    two = torch.sort(kept.abs(), dim=-1, descending=True, stable=True).indices[..., :2]
    D = torch.zeros_like(P).scatter_(3, cols.gather(3, two), kept.gather(3, two))
    return D.reshape(R * V, B * M)[:out, :inn]


def exact(case, seed):
    """Products in fp64.  What is defined to the bit (pruning, merging, the search) has no rounding to measure."""
    g = _generator(seed)
    if case["kind"] == "layer":
        W = _masked64(_weight(g, case["out"], case["in"]), case["V"], case["M"])
        x = _activations(g, case["tokens"], case["in"]).double()
        bias = torch.randn(case["out"], generator=g, device=DEV).to(torch.float16) if case["bias"] else None
        perm = {p: torch.randperm(n, generator=g, device=DEV) if case[p] else None
                for p, n in (("perm_in", case["in"]), ("perm_out", case["out"]))}
        y = (x if perm["perm_in"] is None else x[:, perm["perm_in"]]) @ W.t()
        if bias is not None:
            y += bias.double()
        if perm["perm_out"] is None:
            return y
        z = torch.empty_like(y)
        z[:, perm["perm_out"]] = y
        return z
    if case["kind"] != "block":
        return None
    layers = _layers(case)
    W = [_masked64(_weight(g, o, i), case["V"], case["M"]) for _, o, i, _ in layers]
    widths = {x: i for _, _, i, x in layers}
    xs = [_activations(g, case["tokens"], widths[k]).double() for k in range(len(widths))]
    bias = [torch.randn(o, generator=g, device=DEV).to(torch.float16) if case["bias"] else None for _, o, _, _ in layers]
    return [xs[x] @ w.t() if b is None else xs[x] @ w.t() + b.double() for (_, _, _, x), w, b in zip(layers, W, bias)]
