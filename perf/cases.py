"""Performance cases of the sliced-linear library: what a program that serves, loads or quantises a
model asks of it, through the public binding.

Kinds of case
  linear   one mq_linear / mq_linear_bf16 / mq_linear_from_parent call (N x K layer, M activation rows)
  stack    one mq_linear_stack call over all linears of `blocks` decoder blocks, each with its own width
  decode   one HIP-graph replay of `blocks` decoder blocks in the shape of a decode step: q/k/v in one
           launch, o, gate/up in one launch, down
  load     prepare_layer: slice, pack and re-tile the scales of one layer from its 8-bit parent
  reslice  one mq_reslice_many call: all linears of `blocks` resident decoder blocks to other widths
  quant    one mq_quant_matgptq call over a whole layer
  gptq     one mq_matgptq_quantize call (the working copy of the weights is refreshed first, as the call
           overwrites it)
"""
import math

import torch

import paper_2602_03537_amd as mq
from paper_2602_03537_amd import synth

GROUP = 128
DEVICE = "cuda"
WIDTHS = (2, 3, 4, 6, 8)

# hidden size, key/value size and feed-forward size of the decoder blocks
BLOCK_7B = {"hidden": 4096, "kv": 4096, "ffn": 11008}
BLOCK_70B = {"hidden": 8192, "kv": 1024, "ffn": 28672}


def _linear(N, K, M, r, dtype="fp16", symmetric=False, from_parent=False):
    return {"kind": "linear", "N": N, "K": K, "M": M, "r": r, "dtype": dtype, "symmetric": symmetric,
            "from_parent": from_parent}


def listed():
    return [
        # one projection of a small decoder at batch 1: the smallest call, latency and launch count
        {"name": "linear-4096-m1", **_linear(4096, 4096, 1, 4)},
        # the largest feed-forward projection at batch 1: a single call that is bound by memory
        {"name": "linear-up-m1", **_linear(28672, 8192, 1, 3, symmetric=True)},
        # ragged output size, bf16, a handful of sequences
        {"name": "linear-ragged-bf16-m3", **_linear(13003, 5120, 3, 6, dtype="bf16")},
        # small-batch decoding
        {"name": "linear-up-m16", **_linear(28672, 8192, 16, 4)},
        # medium batch, the long contraction of the down projection
        {"name": "linear-down-m61", **_linear(8192, 28672, 61, 3)},
        # the largest batch a call takes (a prefill chunk)
        {"name": "linear-up-m256", **_linear(28672, 8192, 256, 4)},
        # a whole model's linears at batch 1, widths mixed
        {"name": "stack-7b-m1", "kind": "stack", **BLOCK_7B, "blocks": 32, "M": 1, "bits": 3.5, "pick": 0},
        # large-model blocks at a small batch
        {"name": "stack-70b-m8", "kind": "stack", **BLOCK_70B, "blocks": 4, "M": 8, "bits": 4.0, "pick": 0},
        # decode step: the launches of four blocks in a graph
        {"name": "decode-7b-m1", "kind": "decode", **BLOCK_7B, "blocks": 4, "M": 1, "bits": 3.5, "pick": 0},
        # a resident model changes its width budget
        {"name": "reslice-7b", "kind": "reslice", **BLOCK_7B, "blocks": 4, "bits": 3.5, "pick": 0},
        # the code choice of a whole layer (widths of the method's own experiments)
        {"name": "quant-4096", "kind": "quant", "N": 4096, "K": 4096, "widths": "3,4,8"},
        # the column loop of a whole layer
        {"name": "gptq-4096", "kind": "gptq", "N": 4096, "K": 4096, "widths": "3,4,8", "block": 128},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _most_rows(weights, M):
    """M, or as many rows as keep the products of a pass at those of the largest listed call."""
    return max(1, min(M, 256 * 28672 * 8192 // weights))


def draw(rng):
    kind = rng.choices(("linear", "stack", "decode", "load", "reslice", "quant", "gptq"), (10, 3, 2, 2, 1, 2, 1))[0]
    if kind == "linear":
        N, K = _log(rng, 1000, 28672), 128 * _log(rng, 8, 224)
        c = _linear(N, K, _most_rows(N * K, _log(rng, 1, 256)), rng.choice(WIDTHS), rng.choice(("fp16", "fp16", "bf16")),
                    rng.random() < 0.3)
        if c["M"] <= 4 and c["dtype"] == "fp16":
            c["from_parent"] = rng.random() < 0.25
        return c
    if kind in ("stack", "decode", "reslice"):
        c = {"kind": kind, "hidden": 128 * _log(rng, 16, 64), "kv": 64 * rng.randint(8, 64), "ffn": 128 * _log(rng, 40, 224),
             "blocks": rng.randint(2, 6), "bits": rng.choice((3.5, 4.0)), "pick": rng.randrange(1000)}
        if kind == "stack":
            c["M"] = _most_rows(c["blocks"] * sum(n * k for n, k in _shapes(c)), _log(rng, 1, 96))
        elif kind == "decode":
            c["M"] = rng.randint(1, 4)
        return c
    if kind == "load":
        return {"kind": "load", "N": _log(rng, 1000, 28672), "K": 128 * _log(rng, 8, 224), "r": rng.choice(WIDTHS),
                "symmetric": rng.random() < 0.3}
    widths = rng.choice(("3,4,8", "3,4,8", "2,3,4,6,8", "8", "4,8", "1,2,8"))
    if kind == "quant":
        return {"kind": "quant", "N": _log(rng, 500, 11008), "K": 128 * _log(rng, 4, 64), "widths": widths}
    return {"kind": "gptq", "N": _log(rng, 500, 4096), "K": 128 * _log(rng, 4, 32), "widths": widths,
            "block": rng.choice((64, 128))}


# ------------------------------------------------------------------------------------------ inputs
def _shapes(c):
    h, kv, f = c["hidden"], c["kv"], c["ffn"]
    return [(h, h), (kv, h), (kv, h), (h, h), (f, h), (f, h), (h, f)]


def _layer_list(c):
    """[(N, K, r)] of a case's layers."""
    if "blocks" not in c:
        return [(c["N"], c["K"], c.get("r", 8))]
    shapes = _shapes(c) * c["blocks"]
    bits, _ = synth.draw_bitwidths([n * k for n, k in shapes], c["bits"], seed=c["pick"])
    return [(n, k, int(r)) for (n, k), r in zip(shapes, bits)]


def _gen(seed, i):
    g = torch.Generator(device=DEVICE)
    g.manual_seed((int(seed) * 1_000_003 + 7919 * i) % (1 << 62))
    return g


def _parent(N, K, seed, i, symmetric=False):
    """8-bit parent of Gaussian weights: min-max per group, or symmetric about code 128."""
    if not symmetric:
        L = synth.make_layer_device(N, K, seed=(int(seed) * 1_000_003 + 7919 * i) % (1 << 62), device=DEVICE, want_x=False)
        return L["parent"], L["scales"], L["zeros"]
    G = K // GROUP
    g = _gen(seed, i)
    parent = torch.empty((N, K), dtype=torch.uint8, device=DEVICE)
    scales = torch.empty((N, G), dtype=torch.float16, device=DEVICE)
    rows = max(1, (1 << 26) // K)
    for a in range(0, N, rows):
        b = min(N, a + rows)
        W = torch.randn((b - a, G, GROUP), generator=g, device=DEVICE) * 0.02
        s = (W.abs().amax(dim=2) / 127.0).to(torch.float16)
        q = torch.clamp(torch.round(W / s.float()[:, :, None]) + 128.0, 0, 255)
        parent[a:b] = q.to(torch.uint8).reshape(b - a, K)
        scales[a:b] = s
    return parent, scales, None


def _x(M, K, seed, i, dtype="fp16"):
    x = torch.randn((M, K), generator=_gen(seed, 500_000 + i), device=DEVICE)
    return x.to(torch.bfloat16 if dtype == "bf16" else torch.float16)


def _launches(c):
    """Groups of layer indices that share their activations (one launch each) of a decode step."""
    out = []
    for b in range(c["blocks"]):
        o = 7 * b
        out += [(o, o + 1, o + 2), (o + 3,), (o + 4, o + 5), (o + 6,)]
    return out


def _x_of(c, i):
    """Which activations layer i of a case with blocks reads: q/k/v share theirs, and so do gate/up."""
    return (0, 0, 0, 3, 4, 4, 6)[i % 7] + 7 * (i // 7)


def _weights(c, seed):
    """fp32 weights of a layer and the fixed min-max grid of its groups."""
    N, K = c["N"], c["K"]
    G = K // GROUP
    W = torch.randn((N, K), generator=_gen(seed, 0), device=DEVICE) * 0.02
    lo, hi = W.view(N, G, GROUP).amin(dim=2), W.view(N, G, GROUP).amax(dim=2)
    s = ((hi - lo) / 255.0).to(torch.float16)
    z = torch.clamp(torch.round(-lo / s.float()), 0, 255).to(torch.float16)
    return W, s, z


def _factor(K, seed):
    """Upper Cholesky factor of the inverse Hessian of 2 K correlated Gaussian features of uneven scale."""
    g = _gen(seed, 900_000)
    X = torch.randn((K, 2 * K), generator=g, device=DEVICE)
    X = X * (1.0 + 3.0 * torch.rand((K, 1), generator=g, device=DEVICE))
    X = X + 0.5 * X.roll(1, dims=0)
    H = (X @ X.T) * (2.0 / X.shape[1])
    H.diagonal().add_(0.01 * H.diagonal().mean())
    L = torch.linalg.cholesky(H)
    Li = torch.linalg.solve_triangular(L, torch.eye(K, device=DEVICE), upper=False)
    return torch.linalg.cholesky(Li.T @ Li).T.contiguous()


def prepare(case, seed):
    c = case
    kind = c["kind"]
    if kind == "linear":
        N, K, M, r = c["N"], c["K"], c["M"], c["r"]
        parent, s, z = _parent(N, K, seed, 0, c["symmetric"])
        L = mq.prepare_layer(parent, s, z, 8 if c["from_parent"] else r)
        dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float16
        call = mq.mq_linear_from_parent if c["from_parent"] else mq.mq_linear_bf16 if c["dtype"] == "bf16" else mq.mq_linear
        return {"kind": kind, "call": call, "L": L, "r": r, "x": _x(M, K, seed, 0, c["dtype"]),
                "y": torch.empty((M, N), dtype=dt, device=DEVICE),
                "ws": mq.new_workspace(M, N, K, 8 if c["from_parent"] else r, DEVICE)}
    if kind in ("stack", "decode"):
        M, todo = c["M"], _layer_list(c)
        y = torch.empty(M * sum(n for n, _, _ in todo), dtype=torch.float16, device=DEVICE)
        xs, layers, at = {}, [], 0
        for i, (N, K, r) in enumerate(todo):
            L = mq.prepare_layer(*_parent(N, K, seed, i), r)
            j = _x_of(c, i)
            if j not in xs:
                xs[j] = _x(M, K, seed, j)
            layers.append(dict(L, x=xs[j], y=y[at:at + M * N].view(M, N)))
            at += M * N
        state = {"kind": kind, "layers": layers, "y": y}
        if kind == "stack":
            state["plan"] = mq.mq_stack_plan(layers, M, device=DEVICE)
            return state
        calls = []
        for group in _launches(c):
            if len(group) > 1:
                calls.append((mq.mq_stack_plan([layers[i] for i in group], M, device=DEVICE), None, None))
            else:
                L = layers[group[0]]
                calls.append((None, L, mq.new_workspace(M, L["N"], L["K"], L["r"], DEVICE)))

        def step():
            for plan, L, ws in calls:
                if plan is not None:
                    mq.mq_linear_stack(plan)
                else:
                    mq.mq_linear(L["x"], L["packed_W"], L["scales_t"], L["zeros_t"], L["N"], L["K"], L["r"], GROUP, ws, L["y"])

        step()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        state.update(calls=calls, graph=graph)
        return state
    if kind == "load":
        parent, s, z = _parent(c["N"], c["K"], seed, 0, c["symmetric"])
        return {"kind": kind, "parent": parent, "s": s, "z": z, "r": c["r"]}
    if kind == "reslice":
        todo = _layer_list(c)
        out = torch.empty(sum(mq.mq_packed_bytes(n, k, r) for n, k, r in todo), dtype=torch.uint8, device=DEVICE)
        jobs, at = [], 0
        for i, (N, K, r) in enumerate(todo):
            nb = mq.mq_packed_bytes(N, K, r)
            jobs.append({"packed_parent": mq.mq_pack(_parent(N, K, seed, i)[0], 8, 8), "N": N, "K": K, "r": r,
                         "out": out[at:at + nb]})
            at += nb
        return {"kind": kind, "jobs": jobs, "out": out}
    W, s, z = _weights(c, seed)
    widths = [int(r) for r in c["widths"].split(",")]
    state = {"kind": kind, "W": W, "s": s, "z": z, "widths": widths, "lam": [1.0] * len(widths),
             "Q": torch.empty(W.shape, dtype=torch.uint8, device=DEVICE)}
    if kind == "gptq":
        state.update(U=_factor(c["K"], seed), work=torch.empty_like(W), block=c["block"])
    return state


def run(state):
    kind = state["kind"]
    if kind == "linear":
        L = state["L"]
        return state["call"](state["x"], L["packed_W"], L["scales_t"], L["zeros_t"], L["N"], L["K"], state["r"], GROUP,
                             state["ws"], state["y"])
    if kind == "stack":
        mq.mq_linear_stack(state["plan"])
        return state["y"]
    if kind == "decode":
        state["graph"].replay()
        return state["y"]
    if kind == "load":
        L = mq.prepare_layer(state["parent"], state["s"], state["z"], state["r"])
        return [L["packed_W"], L["scales_t"]] + ([] if L["zeros_t"] is None else [L["zeros_t"]])
    if kind == "reslice":
        mq.mq_reslice_many(state["jobs"])
        return state["out"]
    if kind == "quant":
        return mq.mq_quant_matgptq(state["W"], state["s"], state["z"], state["widths"], state["lam"], out=state["Q"])
    state["work"].copy_(state["W"])
    return mq.mq_matgptq_quantize(state["work"], state["U"], state["s"], state["z"], state["widths"], state["lam"],
                                  block=state["block"], out=state["Q"])


# ------------------------------------------------------------------------------------------ what a pass needs
def _pad(N):
    return (N + 63) // 64 * 64


def work(case):
    c = case
    kind = c["kind"]
    if kind in ("linear", "stack", "decode"):
        M, todo = c["M"], _layer_list(c)
        zeros = 0 if c.get("symmetric") else 1
        by = fl = 0
        for i, (N, K, r) in enumerate(todo):
            bits = 8 if c.get("from_parent") else r
            by += N * K * bits / 8 + (1 + zeros) * 2 * N * K / GROUP + 2 * M * N
            if "blocks" not in c or _x_of(c, i) == i:
                by += 2 * M * K
            fl += 2 * M * N * K
        return {"bytes": by, "flops": fl}
    if kind == "load":
        N, K, r = c["N"], c["K"], c["r"]
        meta = (1 if c["symmetric"] else 2) * 2 * K / GROUP
        return {"bytes": N * K + _pad(N) * K * r / 8 + meta * (N + _pad(N)), "flops": 0}
    if kind == "reslice":
        return {"bytes": sum(_pad(N) * K * (8 + r) / 8 for N, K, r in _layer_list(c)), "flops": 0}
    N, K, R = c["N"], c["K"], len(c["widths"].split(","))
    meta = 4 * N * K / GROUP
    choose = 6.0 * R * N * K  # one candidate per weight and width; what a search adds is the kernel's choice
    if kind == "quant":
        return {"bytes": 5 * N * K + meta, "flops": choose}
    # the copy, the read and the codes; the upper triangle; one multiply and one subtract per (row, column, later column)
    return {"bytes": 4 * N * K * 3 + N * K + meta + 2 * K * K, "flops": choose + float(N) * K * (K - 1)}


def tolerance(case):
    if case["kind"] not in ("linear", "stack", "decode"):
        return "exact"
    # The result is rounded to fp16 (2^-11 at most, 2.1e-4 in the 2-norm) or bf16 (1.7e-3); up to 16 rows products are
    # exact in fp32, above them the weights are rounded to fp16 operands, which adds half as much again.
    if case.get("dtype") == "bf16":
        return {"rel": 7e-3}
    return {"rel": 9e-4 if case["M"] <= 16 else 1.2e-3}


# ------------------------------------------------------------------------------------------ 64-bit results
def _dense64(x, parent, s, z, r):
    """x @ W^T in float64, W the affine de-quantisation of the parent's r-bit slice (round half up, clamp)."""
    N, K = parent.shape
    out = torch.empty((x.shape[0], N), dtype=torch.float64, device=DEVICE)
    x = x.double()
    rows = max(1, (1 << 26) // K)
    for a in range(0, N, rows):
        q = parent[a:a + rows].int()
        t = q if r == 8 else torch.clamp((q + (1 << (7 - r))) >> (8 - r), max=(1 << r) - 1) << (8 - r)
        w = t.double().view(q.shape[0], K // GROUP, GROUP)
        w = w - (128.0 if z is None else z[a:a + rows].double()[:, :, None])
        w = (w * s[a:a + rows].double()[:, :, None]).view(q.shape[0], K)
        out[:, a:a + rows] = x @ w.T
    return out


def exact(case, seed):
    c = case
    if c["kind"] == "linear":
        x = _x(c["M"], c["K"], seed, 0, c["dtype"])
        return _dense64(x, *_parent(c["N"], c["K"], seed, 0, c["symmetric"]), c["r"])
    if c["kind"] in ("stack", "decode"):
        out = []
        for i, (N, K, r) in enumerate(_layer_list(c)):
            out.append(_dense64(_x(c["M"], K, seed, _x_of(c, i)), *_parent(N, K, seed, i), r).reshape(-1))
        return torch.cat(out)
    return None  # codes and packed bytes: whole numbers, compared as they are
