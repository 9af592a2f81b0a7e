"""What the speed of this framework is measured on.

Tree verification with a target model and tree generation with a draft model,
through the calls that a serving loop makes.  A loop keeps its weights in the
kernels' own layout, its caches, its workspace and one HIP graph per call
sequence (the prefix length and the tree live in device memory, so one graph
serves every step); single operations are called eagerly.

Shapes are those of the Llama-3 models that the repository's workloads name:
1b, 8b, 70b, and 70b4, one GPU's share of the 70b layer at tensor parallelism
4.  Trees have 1 to 64 nodes, prefixes 16 to 32768 tokens, and the caches room
for more than the prefix that is in them.
"""
import math

import torch

import paper_2506_11309_amd as ss

THETA = 500000.0
EPS = 1e-5
VOCAB = 128256

SHAPES = {
    "1b": {"H": 2048, "Hq": 32, "Hkv": 8, "D": 64, "F": 8192},
    "8b": {"H": 4096, "Hq": 32, "Hkv": 8, "D": 128, "F": 14336},
    "70b": {"H": 8192, "Hq": 64, "Hkv": 8, "D": 128, "F": 28672},
    "70b4": {"H": 8192, "Hq": 16, "Hkv": 2, "D": 128, "F": 7168},
}


def listed():
    return [
        # one decoder layer of the target model verifying a draft tree, from a graph:
        # a small model and a small tree at a short prefix, where latency and launches count
        {"name": "layer 1b T8", "kind": "layer", "shape": "1b", "T": 8, "P": 512, "S": 2048},
        # a middle-sized model, a tree and a prefix of no round size
        {"name": "layer 8b T13", "kind": "layer", "shape": "8b", "T": 13, "P": 2053, "S": 4096},
        # one GPU's share of a large model at a batch of 8
        {"name": "layer 70b4 T8", "kind": "layer", "shape": "70b4", "T": 8, "P": 1000, "S": 4096},
        # the large model with the tree size that it is mostly run with
        {"name": "layer 70b T32", "kind": "layer", "shape": "70b", "T": 32, "P": 4096, "S": 8192},
        # the largest tree: long context at a middle-sized model, and the large model
        {"name": "layer 8b T64 long", "kind": "layer", "shape": "8b", "T": 64, "P": 32768, "S": 40960},
        {"name": "layer 70b T64", "kind": "layer", "shape": "70b", "T": 64, "P": 8192, "S": 16384},
        # a whole verification forward: 16 layers and the LM head, from a graph
        {"name": "step 1b T8", "kind": "step", "shape": "1b", "layers": 16, "T": 8, "P": 1024, "S": 2048, "V": VOCAB},
        # the MLP block's first half at a tree size between the tile sizes, called eagerly
        {"name": "swiglu 70b T45", "kind": "swiglu", "K": 8192, "N": 28672, "M": 45},
        # final norm and LM head of the large model
        {"name": "head 70b T64", "kind": "head", "H": 8192, "V": VOCAB, "M": 64},
        # one draft expansion's attention, all 16 layers, from a graph
        {"name": "draft attention 1b", "kind": "draft", "shape": "1b", "layers": 16, "w": 8, "N": 56, "P": 4096, "S": 8192},
        # the children of the expanded leaves from the draft model's logits, called eagerly
        {"name": "expand w8", "kind": "expand", "n": 8, "V": VOCAB, "k": 8},
        # closing a step: greedy acceptance and the commit of the accepted path in all layers, from a graph
        {"name": "close 70b T64", "kind": "close", "T": 64, "V": VOCAB, "layers": 80, "Hkv": 8, "D": 128, "P": 700, "S": 1024},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "step", "gemm", "swiglu", "attention", "head", "draft", "expand", "close"])
    T = rng.randint(1, 64)
    P = _log(rng, 16, 32768)
    S = P + T + rng.randint(0, P)
    shape = rng.choice(sorted(SHAPES))
    if kind in ("layer", "attention"):
        return {"kind": kind, "shape": shape, "T": T, "P": P, "S": S}
    if kind == "step":
        P = _log(rng, 16, 4096)
        return {"kind": kind, "shape": rng.choice(["1b", "8b"]), "layers": rng.randint(2, 6), "T": T, "P": P,
                "S": P + T + rng.randint(0, P), "V": 16 * _log(rng, 512, VOCAB // 16)}
    if kind == "gemm":
        return {"kind": kind, "K": 128 * _log(rng, 8, 224), "N": 64 * _log(rng, 16, 512), "M": T, "residual": rng.random() < 0.7}
    if kind == "swiglu":
        return {"kind": kind, "K": 128 * _log(rng, 8, 64), "N": 64 * _log(rng, 16, 448), "M": T}
    if kind == "head":
        return {"kind": kind, "H": 128 * _log(rng, 8, 64), "V": 16 * _log(rng, 512, VOCAB // 16), "M": T}
    if kind == "draft":
        N = rng.randint(0, 64)
        w = _log(rng, 1, 64)
        return {"kind": kind, "shape": rng.choice(["1b", "8b"]), "layers": rng.randint(4, 16), "w": w, "N": N,
                "P": _log(rng, 16, 8192), "S": 8192 + 128 + rng.randint(0, 2048)}
    if kind == "expand":
        return {"kind": kind, "n": _log(rng, 1, 64), "V": _log(rng, 1000, 200000), "k": rng.randint(1, 8)}
    return {"kind": kind, "T": T, "V": _log(rng, 1000, 200000), "layers": rng.randint(4, 80), "Hkv": rng.choice([2, 8]),
            "D": rng.choice([64, 128]), "P": rng.randint(16, 900), "S": 1024}


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        case = _draw(rng)
        if _cost(case) <= most:
            return case


# ------------------------------------------------------------------ inputs


class _Inputs:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, *shape, mean=0.0, std=1.0):
        """fp16 N(mean, std), drawn in pieces so that a cache or an LM head needs no float copy of itself."""
        out = torch.empty(shape, dtype=torch.float16, device="cuda")
        flat = out.view(-1)
        for i in range(0, flat.numel(), 1 << 26):
            n = min(1 << 26, flat.numel() - i)
            flat[i:i + n] = torch.randn(n, generator=self.g, device="cuda") * std + mean
        return out

    def ints(self, hi, *shape):
        return torch.randint(hi, shape, generator=self.g, device="cuda")

    def tree(self, T):
        """Parents of a tree whose nodes hang below one of the (up to 8) nodes before them."""
        u = torch.rand(T, generator=self.g, device="cuda").tolist()
        return [-1] + [i - 1 - int(u[i] * min(i, 8)) for i in range(1, T)]

    def int4(self, K, N):
        """An int4 matrix: N(0, 0.02) weights, quantised by minimum and maximum of each row's groups of 128."""
        q = torch.empty((N, K // 2), dtype=torch.uint8, device="cuda")
        s = torch.empty((N, K // 128), dtype=torch.float16, device="cuda")
        z = torch.empty((N, K // 128), dtype=torch.uint8, device="cuda")
        rows = max(1, (1 << 26) // K)
        for r in range(0, N, rows):
            n = min(rows, N - r)
            w = (torch.randn((n, K // 128, 128), generator=self.g, device="cuda") * 0.02)
            lo, hi = w.amin(-1), w.amax(-1)
            sc = ((hi - lo) / 15).half()
            sf = sc.float()
            zp = torch.round(-lo / sf).clamp_(0, 15)
            qq = (torch.round(w / sf[..., None]) + zp[..., None]).clamp_(0, 15).to(torch.uint8).view(n, K)
            q[r:r + n] = qq[:, 0::2] | (qq[:, 1::2] << 4)
            s[r:r + n] = sc
            z[r:r + n] = zp.to(torch.uint8)
        return {"q": q, "s": s, "z": z}


def _gpu_int32(v):
    return torch.tensor(v, dtype=torch.int32, device="cuda")


def _rope(S, D):
    a = torch.arange(S, device="cuda", dtype=torch.float64)[:, None] * THETA ** (
        -torch.arange(D // 2, device="cuda", dtype=torch.float64) * 2 / D)
    return torch.stack((a.cos(), a.sin()), -1).float().contiguous()


def _caches(x, n, Hkv, S, D, rows):
    """K and V of n layers, [n][Hkv][S][D]; the first `rows` rows drawn."""
    out = []
    for _ in range(2):
        c = torch.zeros((n, Hkv, S, D), dtype=torch.float16, device="cuda")
        for i in range(n):
            c[i, :, :rows] = x.normal(Hkv, rows, D)
        out.append(c)
    return out


def _layer_inputs(x, m, n):
    names = (("wqkv", m["H"], (m["Hq"] + 2 * m["Hkv"]) * m["D"]), ("wo", m["Hq"] * m["D"], m["H"]), ("wgate", m["H"], m["F"]),
             ("wup", m["H"], m["F"]), ("wdown", m["F"], m["H"]))
    out = []
    for _ in range(n):
        layer = {name: x.int4(K, N) for name, K, N in names}
        layer["attn_norm"] = x.normal(m["H"], mean=1.0, std=0.02)
        layer["mlp_norm"] = x.normal(m["H"], mean=1.0, std=0.02)
        out.append(layer)
    return out


def _inputs(case, seed):
    """Everything that is drawn, in the library's public layouts."""
    x, kind = _Inputs(seed), case["kind"]
    if kind in ("layer", "step"):
        m, T, n = SHAPES[case["shape"]], case["T"], case.get("layers", 1)
        d = {"layers": _layer_inputs(x, m, n), "x": x.normal(T, m["H"]), "parent": x.tree(T)}
        d["k"], d["v"] = _caches(x, n, m["Hkv"], case["S"], m["D"], case["P"])
        if kind == "step":
            d["norm"] = x.normal(m["H"], mean=1.0, std=0.02)
            d["head"] = x.normal(case["V"], m["H"], std=0.02)
        return d
    if kind in ("gemm", "swiglu"):
        d = {"w": x.int4(case["K"], case["N"]), "x": x.normal(case["M"], case["K"])}
        if kind == "swiglu":
            d["up"] = x.int4(case["K"], case["N"])
            d["norm"] = x.normal(case["K"], mean=1.0, std=0.02)
        elif case["residual"]:
            d["res"] = x.normal(case["M"], case["N"])
        return d
    if kind == "attention":
        m, T = SHAPES[case["shape"]], case["T"]
        d = {"qkv": x.normal(T, (m["Hq"] + 2 * m["Hkv"]) * m["D"]), "parent": x.tree(T)}
        d["k"], d["v"] = _caches(x, 1, m["Hkv"], case["S"], m["D"], case["P"])
        return d
    if kind == "head":
        return {"x": x.normal(case["M"], case["H"]), "norm": x.normal(case["H"], mean=1.0, std=0.02),
                "head": x.normal(case["V"], case["H"], std=0.02)}
    if kind == "draft":
        m, w, N = SHAPES[case["shape"]], case["w"], case["N"]
        d = {"qkv": x.normal(case["layers"], w, (m["Hq"] + 2 * m["Hkv"]) * m["D"])}
        d["k"], d["v"] = _caches(x, case["layers"], m["Hkv"], case["S"], m["D"], case["P"] + N)
        forest = x.tree(N + 1)  # a tree of N + 1 nodes without its root: a forest below the last prefix token
        d["forest"] = [p - 1 for p in forest[1:]]
        d["leaf"] = (x.ints(N + 1, w) - 1).tolist()
        return d
    if kind == "expand":
        return {"logits": x.normal(case["n"], -(-case["V"] // 8) * 8, std=3.0)}
    T, V = case["T"], case["V"]  # close
    d = {"logits": x.normal(T, -(-V // 8) * 8, std=3.0), "parent": x.tree(T)}
    d["k"], d["v"] = _caches(x, case["layers"], case["Hkv"], case["S"], case["D"], case["P"] + T)
    tokens = x.ints(V, T).tolist()
    best = d["logits"][:, :V].argmax(-1).tolist()
    node = T - 1  # the target agrees with the draft on the way to the last node's parent
    path = []
    while node >= 0:
        path.append(node)
        node = d["parent"][node]
    for child in path[1:-1]:
        tokens[child] = best[d["parent"][child]]
    d["tokens"] = tokens
    return d


# ------------------------------------------------------------------- state


def _w4(w):
    W = ss.make_w4(w["q"], w["s"], w["z"])
    keep = ss.prepack_w4(W)
    return W, keep


def _captured(call):
    g, side = ss.Graph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        g.begin(side)
        call()
        g.end(side)
    torch.cuda.synchronize()
    return g


def prepare(case, seed):
    d, kind, s = _inputs(case, seed), case["kind"], {}
    s["kind"], s["keep"] = kind, d
    if kind in ("layer", "step"):
        m, T, P = SHAPES[case["shape"]], case["T"], case["P"]
        dims = ss.make_dims(m["H"], m["Hq"], m["Hkv"], m["D"], m["F"], case["S"], EPS, THETA)
        packed, layers = [], []
        for i, w in enumerate(d["layers"]):
            mats = []
            for name in ("wqkv", "wo", "wgate", "wup", "wdown"):
                W, keep = _w4(w[name])
                w[name] = None  # the kernels read the packed copy alone
                mats.append(W)
                packed.append(keep)
            layers.append(ss.make_layer(w["attn_norm"], w["mlp_norm"], *mats, d["k"][i], d["v"][i]))
        s["packed"], s["x"], s["hidden"] = packed, d["x"], torch.empty_like(d["x"])
        s["prefix"], s["parent"], s["rope"] = _gpu_int32([P]), _gpu_int32(d["parent"]), _rope(case["S"], m["D"])
        rows_k, rows_v = d["k"][:, :, P:P + T], d["v"][:, :, P:P + T]
        if kind == "layer":
            s["ws"] = ss.workspace(ss.verify_layer_workspace_bytes(dims, T))
            s["out"] = [s["hidden"], rows_k, rows_v]
            s["graph"] = _captured(lambda: ss.verify_layer(layers[0], dims, s["hidden"], s["prefix"], s["parent"], s["rope"], s["ws"]))
        else:
            logits = torch.empty((T, case["V"]), dtype=torch.float16, device="cuda")
            s["ws"] = ss.workspace(ss.verify_step_workspace_bytes(dims, T, case["V"]))
            s["out"] = [logits, s["hidden"], rows_k, rows_v]
            array = ss.make_layers(layers)
            s["graph"] = _captured(lambda: ss.verify_step(array, dims, s["hidden"], s["prefix"], s["parent"], s["rope"], s["ws"],
                                                          d["norm"], d["head"], logits))
    elif kind in ("gemm", "swiglu"):
        s["W"], s["packed"] = _w4(d["w"])
        s["x"], s["norm"], s["res"] = d["x"], d.get("norm"), d.get("res")
        s["y"] = torch.empty((case["M"], case["N"]), dtype=torch.float16, device="cuda")
        if kind == "swiglu":
            s["up"], s["packed_up"] = _w4(d["up"])
            s["ws"] = ss.workspace(ss.swiglu_workspace_bytes(case["M"], case["K"], case["N"]))
        else:
            s["ws"] = ss.workspace(ss.gemm_workspace_bytes(case["M"], case["K"], case["N"]))
    elif kind == "attention":
        m, T, P = SHAPES[case["shape"]], case["T"], case["P"]
        nq, nkv = m["Hq"] * m["D"], m["Hkv"] * m["D"]
        s["m"], s["q"], s["k"], s["v"] = m, d["qkv"][:, :nq], d["qkv"][:, nq:nq + nkv], d["qkv"][:, nq + nkv:]
        s["kc"], s["vc"] = d["k"][0], d["v"][0]
        s["prefix"], s["parent"], s["rope"] = _gpu_int32([P]), _gpu_int32(d["parent"]), _rope(case["S"], m["D"])
        s["ws"] = ss.workspace(ss.tree_attention_workspace_bytes(T, m["Hq"], m["Hkv"], m["D"], case["S"]))
        s["o"] = torch.empty((T, nq), dtype=torch.float16, device="cuda")
        s["out"] = [s["o"], s["kc"][:, P:P + T], s["vc"][:, P:P + T]]
    elif kind == "head":
        s["x"], s["norm"], s["head"] = d["x"], d["norm"], d["head"]
        s["ws"] = ss.workspace(ss.lm_head_workspace_bytes(case["M"], case["H"], case["V"]))
        s["logits"] = torch.empty((case["M"], case["V"]), dtype=torch.float16, device="cuda")
    elif kind == "draft":
        m, w, N, P = SHAPES[case["shape"]], case["w"], case["N"], case["P"]
        nq, nkv = m["Hq"] * m["D"], m["Hkv"] * m["D"]
        s["prefix"], s["leaf"], s["rope"] = _gpu_int32([P]), _gpu_int32(d["leaf"]), _rope(case["S"], m["D"])
        s["forest"] = _gpu_int32(d["forest"]) if N else None
        s["ws"] = ss.workspace(ss.tree_attention_workspace_bytes(w, m["Hq"], m["Hkv"], m["D"], case["S"]))
        o = torch.empty((case["layers"], w, nq), dtype=torch.float16, device="cuda")
        s["out"] = [o, d["k"][:, :, P + N:P + N + w], d["v"][:, :, P + N:P + N + w]]

        def all_layers():
            for i in range(case["layers"]):
                q = d["qkv"][i]
                ss.draft_tree_attention(q[:, :nq], q[:, nq:nq + nkv], q[:, nq + nkv:], d["k"][i], d["v"][i], s["prefix"], s["forest"],
                                        s["leaf"], m["Hq"], m["Hkv"], s["rope"], o[i], s["ws"])
        s["graph"] = _captured(all_layers)
    elif kind == "expand":
        n, k = case["n"], case["k"]
        s["logits"], s["V"] = d["logits"], case["V"]
        s["tokens"] = torch.empty((n, k), dtype=torch.int32, device="cuda")
        s["logprobs"] = torch.empty((n, k), dtype=torch.float32, device="cuda")
        s["ws"] = ss.workspace(ss.topk_logprobs_workspace_bytes(n))
    else:
        T, P = case["T"], case["P"]
        s["tokens"], s["parent"], s["prefix"] = _gpu_int32(d["tokens"]), _gpu_int32(d["parent"]), _gpu_int32([P])
        argmax, accepted, bonus, length = (_gpu_int32([0] * n) for n in (T, 1, 1, 1))
        s["ws"] = ss.workspace(ss.greedy_accept_workspace_bytes(T))
        s["out"] = [argmax, accepted, bonus, length, d["k"][:, :, P:P + T], d["v"][:, :, P:P + T]]

        def close():
            ss.greedy_accept(d["logits"], s["tokens"], s["parent"], argmax, accepted, bonus, s["ws"], path_len=length, V=case["V"])
            # the prefix length stays, so that the same call can be made again
            ss.kv_commit(d["k"], d["v"], s["prefix"], s["parent"], accepted, n_layers=case["layers"], ws=s["ws"])
        s["graph"] = _captured(close)
    torch.cuda.synchronize()
    return s


def run(s):
    kind = s["kind"]
    if kind in ("layer", "step"):
        s["hidden"].copy_(s["x"])  # the embeddings of this step's tree tokens
        s["graph"].launch()
        return s["out"]
    if kind in ("draft", "close"):
        s["graph"].launch()
        return s["out"]
    if kind == "gemm":
        ss.w4a16_gemm(s["W"], s["x"], s["y"], s["ws"], residual=s["res"])
        return s["y"]
    if kind == "swiglu":
        ss.rmsnorm_w4a16_swiglu(s["W"], s["up"], s["x"], s["norm"], s["y"], s["ws"], EPS)
        return s["y"]
    if kind == "attention":
        m = s["m"]
        ss.tree_attention(s["q"], s["k"], s["v"], s["kc"], s["vc"], s["prefix"], s["parent"], m["Hq"], m["Hkv"], m["D"], s["rope"],
                          s["o"], s["ws"])
        return s["out"]
    if kind == "head":
        ss.lm_head(s["x"], s["norm"], s["head"], s["logits"], s["ws"], EPS)
        return s["logits"]
    ss.topk_logprobs(s["logits"], s["tokens"], s["logprobs"], s["ws"], V=s["V"])
    return [s["tokens"], s["logprobs"]]


# ------------------------------------------------- work, tolerance, 64 bits


def _w4_work(M, K, N):
    return K * N // 2 + 3 * N * (K // 128), 2 * M * K * N


def _attention_work(m, T, keys):
    nq, nkv = m["Hq"] * m["D"], m["Hkv"] * m["D"]
    return 2 * (2 * nkv * keys + T * (2 * nq + 4 * nkv)), 4 * T * nq * keys


def work(case):
    kind = case["kind"]
    if kind in ("layer", "step"):
        m, T, n = SHAPES[case["shape"]], case["T"], case.get("layers", 1)
        parts = [_w4_work(T, m["H"], (m["Hq"] + 2 * m["Hkv"]) * m["D"]), _w4_work(T, m["Hq"] * m["D"], m["H"]), _w4_work(T, m["H"], 2 * m["F"]),
                 _w4_work(T, m["F"], m["H"]), _attention_work(m, T, case["P"] + T)]
        b, f = n * (sum(p[0] for p in parts) + 4 * m["H"]) + 4 * T * m["H"], n * sum(p[1] for p in parts)
        if kind == "step":
            b, f = b + 2 * case["V"] * (m["H"] + T), f + 2 * T * m["H"] * case["V"]
        return {"bytes": b, "flops": f}
    if kind == "gemm":
        b, f = _w4_work(case["M"], case["K"], case["N"])
        return {"bytes": b + 2 * case["M"] * (case["K"] + case["N"] * (2 if case["residual"] else 1)), "flops": f}
    if kind == "swiglu":
        b, f = _w4_work(case["M"], case["K"], 2 * case["N"])
        return {"bytes": b + 2 * case["M"] * (case["K"] + case["N"]) + 2 * case["K"], "flops": f}
    if kind == "attention":
        b, f = _attention_work(SHAPES[case["shape"]], case["T"], case["P"] + case["T"])
        return {"bytes": b, "flops": f}
    if kind == "head":
        return {"bytes": 2 * (case["V"] * case["H"] + case["M"] * (case["V"] + case["H"])), "flops": 2 * case["M"] * case["V"] * case["H"]}
    if kind == "draft":
        b, f = _attention_work(SHAPES[case["shape"]], case["w"], case["P"] + case["N"] + case["w"])
        return {"bytes": case["layers"] * b, "flops": case["layers"] * f}
    if kind == "expand":
        return {"bytes": 2 * case["n"] * case["V"] + 8 * case["n"] * case["k"], "flops": 4 * case["n"] * case["V"]}
    # a path of about an eighth to a half of the tree moves; T / 4 rows stand for it
    moved = case["layers"] * 2 * case["Hkv"] * max(1, case["T"] // 4) * case["D"] * 2
    return {"bytes": 2 * case["T"] * case["V"] + 2 * moved, "flops": case["T"] * case["V"]}


def tolerance(case):
    kind = case["kind"]
    if kind == "close":
        return "exact"
    if kind == "expand":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    # four times the distance from exact() that was seen: 2.9e-4 (head) and 3.6e-4
    # (swiglu), where the one rounding of the fp16 result is most of it, 4.0e-4 for
    # attention (fp16 queries and partials), up to 1.0e-3 for a layer (five stored
    # fp16 intermediates) and 2.2e-3 for 16 layers and the head
    return {"rel": {"gemm": 1.2e-3, "head": 1.2e-3, "swiglu": 1.5e-3, "attention": 1.6e-3, "draft": 1.6e-3, "layer": 4e-3, "step": 9e-3}[kind]}


def _w64(w):
    """fp64 values of an int4 matrix in its public layout, [N][K]."""
    N, K = w["q"].shape[0], 2 * w["q"].shape[1]
    q = torch.stack((w["q"] & 15, w["q"] >> 4), -1).view(N, K // 128, 128).double()
    return ((q - w["z"].double()[..., None]) * w["s"].double()[..., None]).view(N, K)


def _mul(x, w):
    """x . W^T in fp64, W int4 in its public layout or fp16, a piece of its rows at a time."""
    N = w["q"].shape[0] if isinstance(w, dict) else w.shape[0]
    out = []
    for r in range(0, N, 8192):
        piece = _w64({k: t[r:r + 8192] for k, t in w.items()}) if isinstance(w, dict) else w[r:r + 8192].double()
        out.append(x @ piece.t())
    return torch.cat(out, -1)


def _norm64(x, gamma):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gamma.double()


def _silu64(g):
    return g / (1 + torch.exp(-g))


def _rotate64(x, pos):
    """x [T][h][D] rotated at positions pos [T]."""
    D = x.shape[-1]
    a = pos.double()[:, None] * THETA ** (-torch.arange(D // 2, device=x.device, dtype=torch.float64) * 2 / D)
    c, s = a.cos()[:, None], a.sin()[:, None]
    lo, hi = x[..., :D // 2], x[..., D // 2:]
    return torch.cat((lo * c - hi * s, hi * c + lo * s), -1)


def _root_paths(parent):
    """[n][n] bool: j is i or above it; and the depths."""
    see, depth = [[False] * len(parent) for _ in parent], []
    for i, p in enumerate(parent):
        if p >= 0:
            see[i] = list(see[p])
        see[i][i] = True
        depth.append(depth[p] + 1 if p >= 0 else 0)
    return see, depth


def _attend64(q, k, v, kc, vc, keys, pos, see, m):
    """Queries q over the first `keys` cache rows and the new rows, of which query i sees see[i] ([T][keys + T], bool)."""
    T, D, G = q.shape[0], m["D"], m["Hq"] // m["Hkv"]
    q = _rotate64(q.view(T, m["Hq"], D), pos)
    k, v = _rotate64(k.view(T, m["Hkv"], D), pos), v.view(T, m["Hkv"], D)
    out = []
    for g in range(m["Hkv"]):
        K = torch.cat((kc[g, :keys].double(), k[:, g]))
        V = torch.cat((vc[g, :keys].double(), v[:, g]))
        qq = q[:, g * G:(g + 1) * G].reshape(T * G, D)
        sc = (qq @ K.t()) / math.sqrt(D)
        sc = sc.masked_fill(~see.repeat_interleave(G, 0), -math.inf)
        out.append((torch.softmax(sc, -1) @ V).view(T, G * D))
    return torch.cat(out, -1), k.transpose(0, 1), v.transpose(0, 1)


def _tree_attend64(qkv, kc, vc, case, parent, m):
    T, P, nq, nkv = case["T"], case["P"], m["Hq"] * m["D"], m["Hkv"] * m["D"]
    path, depth = _root_paths(parent)
    see = torch.cat((torch.ones((T, P), dtype=torch.bool), torch.tensor(path)), -1).cuda()
    pos = torch.tensor(depth, device="cuda") + P
    return _attend64(qkv[:, :nq], qkv[:, nq:nq + nkv], qkv[:, nq + nkv:], kc, vc, P, pos, see, m)


def exact(case, seed):
    d, kind = _inputs(case, seed), case["kind"]
    if kind in ("layer", "step"):
        m, h, rows = SHAPES[case["shape"]], d["x"].double(), []
        for i, w in enumerate(d["layers"]):
            o, k, v = _tree_attend64(_mul(_norm64(h, w["attn_norm"]), w["wqkv"]), d["k"][i], d["v"][i], case, d["parent"], m)
            rows.append((k, v))
            h = h + _mul(o, w["wo"])
            n = _norm64(h, w["mlp_norm"])
            h = h + _mul(_silu64(_mul(n, w["wgate"])) * _mul(n, w["wup"]), w["wdown"])
        out = [h, torch.stack([r[0] for r in rows]), torch.stack([r[1] for r in rows])]
        return out if kind == "layer" else [_mul(_norm64(h, d["norm"]), d["head"])] + out
    if kind == "gemm":
        y = _mul(d["x"].double(), d["w"])
        return y + d["res"].double() if case["residual"] else y
    if kind == "swiglu":
        n = _norm64(d["x"].double(), d["norm"])
        return _silu64(_mul(n, d["w"])) * _mul(n, d["up"])
    if kind == "attention":
        return list(_tree_attend64(d["qkv"].double(), d["k"][0], d["v"][0], case, d["parent"], SHAPES[case["shape"]]))
    if kind == "head":
        return _mul(_norm64(d["x"].double(), d["norm"]), d["head"])
    if kind == "draft":
        m, w, N, P = SHAPES[case["shape"]], case["w"], case["N"], case["P"]
        nq, nkv = m["Hq"] * m["D"], m["Hkv"] * m["D"]
        path, depth = _root_paths(d["forest"])
        # a new token sees the prefix, its parent's root path and itself
        cached = torch.tensor([path[p] if p >= 0 else [False] * N for p in d["leaf"]]).view(w, N)
        see = torch.cat((torch.ones((w, P), dtype=torch.bool), cached, torch.eye(w, dtype=torch.bool)), -1).cuda()
        pos = torch.tensor([depth[p] + 1 if p >= 0 else 0 for p in d["leaf"]], device="cuda") + P
        each = [_attend64(q[:, :nq], q[:, nq:nq + nkv], q[:, nq + nkv:], d["k"][i], d["v"][i], P + N, pos, see, m)
                for i, q in enumerate(d["qkv"].double())]
        return [torch.stack([e[j] for e in each]) for j in range(3)]
    if kind == "expand":
        x = d["logits"][:, :case["V"]].double()
        value, token = torch.sort(x, dim=-1, descending=True, stable=True)
        return [token[:, :case["k"]], value[:, :case["k"]] - torch.logsumexp(x, -1, keepdim=True)]
    best = d["logits"][:, :case["V"]].double().max(-1, keepdim=True)[0]
    index = torch.arange(case["V"], device="cuda")
    choice = torch.where(d["logits"][:, :case["V"]].double() == best, index, case["V"]).min(-1)[0].tolist()
    node, path = 0, [0]
    while True:
        node = next((i for i in range(1, case["T"]) if d["parent"][i] == node and d["tokens"][i] == choice[node]), None)
        if node is None:
            break
        path.append(node)
    P, T = case["P"], case["T"]
    rows = []
    for c in (d["k"], d["v"]):
        r = c[:, :, P:P + T].double()
        r[:, :, :len(path)] = c[:, :, [P + i for i in path]].double()
        rows.append(r)
    last = path[-1]
    return [torch.tensor(choice), torch.tensor([last]), torch.tensor([choice[last]]), torch.tensor([len(path)])] + rows
