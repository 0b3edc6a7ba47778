"""Timed cases of the framework: what a program built on it runs, through its public entry points.

A case is a dict of plain values.  `prepare` makes what a program holds before the call (device
tensors, a context, nodes and a program with its contracts, a batch or a model); `run` is one
pass.  Every pass runs with contracts on (mode pre_post, the default).

The kinds, and the options that they take:
  chain      z = (2x + 1) + y, s = sum z with range and sum contracts (plain vs fused benchmark)
  filter     affine, exp(-u^2), product, filter with compaction, sum / max / count, and an int32
             sortedness check (the headline benchmark); interpreter or specialized kernel
  product    C = A B with the probabilistic product postcondition
  sort       quicksort of Listing 3 with its two postconditions, float32 or int32
  transpose  transpose with 'every entry finite'
  matvec     y = M v and z = y M (a power-iteration or least-squares step)
  det        determinant by Gaussian elimination
  batch      many uneven programs in one graph-captured launch, every sum read back
  train      one epoch of the plan selector's cost model
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1410_6685_amd as sg
import workloads as W

STATUS_CODE = {name: code for code, name in sg.STATUS.items()}


# ---- the cases ------------------------------------------------------------------------------------

def listed():
    return [
        # a scalar query on a small collection: launch and host latency
        {"name": "chain_1k", "kind": "chain", "n": 1000},
        # the plain-vs-fused benchmark size: fits the last-level cache
        {"name": "chain_1m", "kind": "chain", "n": 1 << 20},
        # the headline benchmark: run-time compiled kernel on the plan the autotuner finds for it
        {"name": "filter_64m", "kind": "filter", "n": 1 << 26, "specialize": True},
        # matrix product at the benchmark's size, and an ordinary ragged one
        {"name": "product_4096", "kind": "product", "m": 4096, "k": 4096, "n": 4096},
        {"name": "product_ragged", "kind": "product", "m": 1000, "k": 1531, "n": 777},
        # the largest sort the paper plots, and a small one of integers with many ties
        {"name": "sort_100m", "kind": "sort", "n": 10 ** 8, "dtype": "f32"},
        {"name": "sort_200k_i32", "kind": "sort", "n": 200_003, "dtype": "i32"},
        # the largest transpose the paper plots
        {"name": "transpose_10k", "kind": "transpose", "rows": 10_000, "cols": 10_000},
        # vector iteration on a matrix that does not fit the last-level cache
        {"name": "matvec_10k", "kind": "matvec", "rows": 10_000, "cols": 8_192},
        # the largest determinant the paper plots
        {"name": "det_1000", "kind": "det", "n": 1000},
        # uneven programs in one launch, lengths log-uniform
        {"name": "batch_256", "kind": "batch", "count": 256, "lo": 10.0, "hi": 22.0},
        # the selector's training: batches of 128, the last one partial
        {"name": "train_10k", "kind": "train", "n": 10_000, "batch": 128},
    ]


def _log(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]; odd as often as even."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["chain", "chain", "filter", "filter", "product", "product", "sort", "sort", "transpose", "matvec",
                       "det", "batch", "train"])
    if kind == "chain":
        return {"kind": kind, "n": _log(rng, 1, 1 << 26)}
    if kind == "filter":
        n = _log(rng, 1000, 1 << 26)
        return {"kind": kind, "n": n if rng.random() < 0.5 else max(1024, n // 1024 * 1024),
                "specialize": rng.random() < 0.5}
    if kind == "product":
        m, k, n = (_log(rng, 16, 4096) for _ in range(3))
        if rng.random() < 0.5:
            m, k, n = (max(16, v // 16 * 16) for v in (m, k, n))
        return {"kind": kind, "m": m, "k": k, "n": n}
    if kind == "sort":
        return {"kind": kind, "n": _log(rng, 100, 10 ** 8), "dtype": rng.choice(["f32", "i32"])}
    if kind in ("transpose", "matvec"):
        return {"kind": kind, "rows": _log(rng, 100, 10_000), "cols": _log(rng, 100, 10_000 if kind == "transpose" else 8_192)}
    if kind == "det":
        return {"kind": kind, "n": _log(rng, 10, 1000)}
    if kind == "batch":
        lo = rng.uniform(8.0, 12.0)
        return {"kind": kind, "count": _log(rng, 16, 256), "lo": round(lo, 2), "hi": round(rng.uniform(lo + 4.0, 22.0), 2)}
    return {"kind": kind, "n": _log(rng, 500, 10_000), "batch": rng.choice([32, 64, 100, 128])}


# ---- inputs ---------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed * 1009 + 17)


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda")


def _uniform(g, *shape):
    """float32 uniform on [-1, 1)."""
    return torch.rand(*shape, generator=g, device="cuda").mul_(2).sub_(1)


def _keys(g, n):
    """Sorted int32 keys with a tenth of a per cent of the positions exchanged in pairs."""
    k = torch.randint(-(1 << 31), (1 << 31) - 1, (n,), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    k = k.sort().values
    pos = torch.randint(0, n, (2 * (n // 1000),), generator=g, device="cuda").unique()
    half = pos.numel() // 2
    if half:
        pos = pos[torch.randperm(pos.numel(), generator=g, device="cuda")]
        a, b = pos[:half], pos[half:2 * half]
        ka, kb = k[a], k[b]
        k[a], k[b] = kb, ka
    return k


def _inputs(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "chain":
        return {"x": _uniform(g, case["n"]), "y": _uniform(g, case["n"])}
    if kind == "filter":
        return {"x": _normal(g, case["n"]), "y": _normal(g, case["n"]), "keys": _keys(g, case["n"])}
    if kind == "product":
        m, k, n = case["m"], case["k"], case["n"]
        return {"A": _normal(g, m, k).div_(math.sqrt(k)), "B": _normal(g, k, n).div_(math.sqrt(k)), "R": _uniform(g, 4, n)}
    if kind == "sort":
        if case["dtype"] == "f32":
            return {"a": _normal(g, case["n"])}
        return {"a": torch.randint(-case["n"] // 8 - 1, case["n"] // 8 + 1, (case["n"],), generator=g, device="cuda",
                                   dtype=torch.int32)}
    if kind == "transpose":
        return {"M": _normal(g, case["rows"], case["cols"])}
    if kind == "matvec":
        return {"M": _normal(g, case["rows"], case["cols"]).div_(math.sqrt(case["cols"])), "v": _normal(g, case["cols"])}
    if kind == "det":
        return {"A": _normal(g, case["n"], case["n"])}
    if kind == "train":
        X = _normal(g, case["n"], 24)
        w = _normal(g, 24).div_(math.sqrt(24.0))
        return {"X": X, "T": torch.tanh((X * w).sum(1)) + 0.1 * X[:, 0] ** 2}
    raise ValueError(kind)


def _batch_specs(case, seed):
    lengths = W.cfg4_lengths(case["count"], seed, case["lo"], case["hi"])
    return W.cfg4_instances(case["count"], seed, seed * 100_003 + 42, lengths)


def _batch_inputs(specs, seed):
    """Every instance's inputs as views of one device buffer, each 64-element aligned."""
    offs, total = [], 0
    for sp in specs:
        views = {}
        for inp in sp["inputs"]:
            views[inp["name"]] = (total, inp["n"])
            total += (inp["n"] + 63) // 64 * 64
        offs.append(views)
    buf = _uniform(_gen(seed), total)
    return [{name: buf[o:o + n] for name, (o, n) in views.items()} for views in offs]


def _spec(case):
    kind = case["kind"]
    if kind == "chain":
        return W.cfg1_spec(case["n"])
    if kind == "filter":
        return W.cfg2_spec(case["n"])
    if kind == "product":
        m, k, n = case["m"], case["k"], case["n"]
        spec = W.cfg3_spec(n)
        for inp, (r, c) in zip(spec["inputs"], ((m, k), (k, n), (4, n))):
            inp["rows"], inp["cols"] = r, c
        return spec
    if kind == "sort":
        return {"inputs": [{"name": "a", "dtype": case["dtype"], "n": case["n"]}],
                "nodes": [{"name": "r", "op": "qsort", "src": "a"}],
                "contracts": [{"kind": "ensure", "check": "sorted", "node": "r"},
                              {"kind": "ensure", "check": "count_eq", "node": "r", "other": "a"}],
                "outputs": ["r"]}
    M = {"name": "M", "dtype": "f32", "rows": case.get("rows"), "cols": case.get("cols")}
    if kind == "transpose":
        return {"inputs": [M], "nodes": [{"name": "T", "op": "transpose", "src": "M"}],
                "contracts": [{"kind": "ensure", "check": "for_all", "node": "T", "pred": ["isfinite"]}],
                "outputs": ["T"]}
    if kind == "det":
        return {"inputs": [{"name": "A", "dtype": "f32", "rows": case["n"], "cols": case["n"]}],
                "nodes": [{"name": "d", "op": "gauss_det", "src": "A"}], "contracts": [], "outputs": ["d"]}
    raise ValueError(kind)


# ---- one pass -------------------------------------------------------------------------------------

class _View:
    """A computed collection's device memory as a tensor (the node is kept alive with it)."""

    def __init__(self, node, shape=None, typestr="<f4"):
        ptr, n = node.device_ptr()
        self.node = node
        self.__cuda_array_interface__ = {"data": (ptr or 0, False), "shape": shape or (n,), "strides": None,
                                         "typestr": typestr, "version": 2}


def _tensor(node, shape=None, typestr="<f4"):
    return torch.as_tensor(_View(node, shape, typestr), device="cuda")


def _verdicts(status, verdicts):
    """Status and every clause's verdict and index as whole numbers."""
    out = [STATUS_CODE[status]]
    for v in verdicts:
        out += [v.holds, v.first_index]
    return np.array(out, np.int64)


def prepare(case, seed):
    ctx = sg.Context(0)
    state = {"case": case, "ctx": ctx}
    kind = case["kind"]
    if kind == "batch":
        specs = _batch_specs(case, seed)
        views = _batch_inputs(specs, seed)
        state["built"] = [sg.build_spec(ctx, sp, v) for sp, v in zip(specs, views)]
        ctx.set_launch(256, 4)
        ctx.set_batch_substeps(4)
        state["batch"] = sg.Batch(ctx, [b.program for b in state["built"]], use_graph=True)
        return state
    inp = _inputs(case, seed)
    if kind == "train":
        state["net"] = sg.Mlp(ctx, W.mlp_init_params(seed))
        state.update(inp)
        return state
    if kind == "matvec":
        M, v = ctx.wrap(inp["M"]), ctx.wrap(inp["v"])
        state["y"] = M.right_multiply(v)
        state["z"] = M.left_multiply(state["y"])
        state["program"] = sg.Program(ctx)
        state["program"].add_root(state["y"])
        state["program"].add_root(state["z"])
        return state
    if case.get("specialize"):
        ctx.set_specialize(True)
    state["built"] = sg.build_spec(ctx, _spec(case), inp)
    state["program"] = state["built"].program
    if case.get("specialize") and case["n"] >= 1 << 20:
        state["program"].set_plan((256, 4, 2, -1))
    if kind == "filter":
        # the output vector at its capacity, nothing but zeros behind the kept items
        state["program"].execute()
        _tensor(state["built"]["k"], (case["n"],)).zero_()
    return state


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "batch":
        status, verdicts = state["batch"].run()
        return {"sums": np.array([b["s"].scalar()[0] for b in state["built"]], np.float32),
                "verdicts": np.array([(v.holds, v.first_index) for v in verdicts], np.int64),
                "status": np.array([STATUS_CODE[s] for s in status], np.int64)}
    if kind == "train":
        losses = state["net"].train(state["X"], state["T"], batch=case["batch"], epochs=1, lr=1e-3)
        return {"params": state["net"].params(), "losses": losses}
    status, verdicts = state["program"].execute()
    if kind == "matvec":
        return {"y": _tensor(state["y"], (case["rows"],)), "z": _tensor(state["z"], (case["cols"],))}
    nodes, out = state["built"], {"verdicts": _verdicts(status, verdicts)}
    if kind == "chain":
        out["s"], out["shadow"] = np.float32(nodes["s"].scalar()[0]), nodes["s"].shadow()
    elif kind == "filter":
        out["k"] = _tensor(nodes["k"], (case["n"],))
        out["s"], out["shadow"] = np.float32(nodes["s"].scalar()[0]), nodes["s"].shadow()
        out["m"], out["c"] = np.float32(nodes["m"].scalar()[0]), nodes["c"].scalar()[1]
    elif kind == "product":
        out["C"] = _tensor(nodes["C"], (case["m"], case["n"]))
    elif kind == "sort":
        out["r"] = _tensor(nodes["r"], None, "<f4" if case["dtype"] == "f32" else "<i4")
    elif kind == "transpose":
        out["T"] = _tensor(nodes["T"], (case["cols"], case["rows"]))
    elif kind == "det":
        out["sign"], out["mant"], out["expo"] = nodes["d"].det_parts()
    return out


# ---- what a pass cannot do without ----------------------------------------------------------------

def work(case):
    kind, n = case["kind"], case.get("n", 0)
    if kind == "chain":
        return {"bytes": 8.0 * n, "flops": 5.0 * n}
    if kind == "filter":  # about 0.44 of the elements are kept
        return {"bytes": 12.0 * n + 4.0 * 0.36 * n, "flops": 30.0 * n}
    if kind == "product":
        m, k = case["m"], case["k"]
        return {"bytes": 4.0 * (m * k + k * n + m * n + 4 * n), "flops": 2.0 * m * k * n}
    if kind == "sort":
        return {"bytes": 8.0 * n, "flops": 0.0}
    if kind == "transpose":
        return {"bytes": 8.0 * case["rows"] * case["cols"], "flops": 0.0}
    if kind == "matvec":
        r, c = case["rows"], case["cols"]
        return {"bytes": 4.0 * (r * c + r + 2 * c), "flops": 4.0 * r * c}
    if kind == "det":
        return {"bytes": 4.0 * n * n, "flops": 2.0 / 3.0 * n ** 3}
    if kind == "batch":
        mean = (2.0 ** case["hi"] - 2.0 ** case["lo"]) / ((case["hi"] - case["lo"]) * math.log(2.0))
        return {"bytes": 4.0 * 1.5 * mean * case["count"], "flops": 4.0 * mean * case["count"]}
    # forward, both halves of the backward, and the parameters' update of every batch
    steps = math.ceil(n / case["batch"])
    return {"bytes": 4.0 * 25 * n + 4.0 * 6 * 5825, "flops": 6.0 * 5696 * n + 12.0 * 5825 * steps}


# ---- the same in 64 bits --------------------------------------------------------------------------

def _exact_train(case, inp, seed):
    X, T = inp["X"].double().cpu().numpy(), inp["T"].double().cpu().numpy()
    p = W.mlp_init_params(seed).astype(np.float64)
    m, v = np.zeros_like(p), np.zeros_like(p)
    lr, b1, b2, eps = (float(np.float32(c)) for c in (1e-3, 0.9, 0.999, 1e-8))
    cut = np.cumsum([24 * 64, 64, 64 * 64, 64, 64])
    total = 0.0
    for step, s0 in enumerate(range(0, case["n"], case["batch"]), 1):
        x, t = X[s0:s0 + case["batch"]], T[s0:s0 + case["batch"]]
        w1, c1, w2, c2, w3, c3 = np.split(p, cut)
        w1, w2 = w1.reshape(24, 64), w2.reshape(64, 64)
        h1 = np.maximum(x @ w1 + c1, 0)
        h2 = np.maximum(h1 @ w2 + c2, 0)
        e = h2 @ w3 + c3 - t
        total += float((e * e).sum())
        dy = 2 * e / len(t)
        d2 = dy[:, None] * w3 * (h2 > 0)
        d1 = (d2 @ w2.T) * (h1 > 0)
        g = np.concatenate([(x.T @ d1).ravel(), d1.sum(0), (h1.T @ d2).ravel(), d2.sum(0), h2.T @ dy, [dy.sum()]])
        m = b1 * m + (1 - b1) * g
        v = b2 * v + (1 - b2) * g * g
        p = p - lr * (m / (1 - b1 ** step)) / (np.sqrt(v / (1 - b2 ** step)) + eps)
    return {"params": p, "losses": np.array([total / case["n"]])}


def _exact_batch(case, seed):
    """The sums of the chains in 64 bits; a filter keeps what the element-wise float32 chain keeps."""
    specs = _batch_specs(case, seed)
    sums = []
    for sp, views in zip(specs, _batch_inputs(specs, seed)):
        lo, hi = {"x": views["x"]}, {"x": views["x"].double()}
        if "y" in views:
            lo["y"], hi["y"] = views["y"], views["y"].double()
        kept = None
        for nd in sp["nodes"]:
            if nd["op"] == "reduce":
                sums.append(float(hi[nd["src"]].sum()))
                continue
            if nd["op"] == "zip":
                op = torch.add if nd["binop"] == "add" else torch.mul
                b = {"lo": lo["y"], "hi": hi["y"]}
                lo[nd["name"]], hi[nd["name"]] = op(lo[nd["a"]], b["lo"]), op(hi[nd["a"]], b["hi"])
                continue
            a, h = lo[nd["src"]], hi[nd["src"]]
            if nd["op"] == "filter":
                kept = a > nd["pred"][2]
                lo[nd["name"]], hi[nd["name"]] = a[kept], h[kept]
            elif nd["fn"][0] == "affine":
                lo[nd["name"]], hi[nd["name"]] = a * nd["fn"][1] + nd["fn"][2], h * nd["fn"][1] + nd["fn"][2]
            else:
                lo[nd["name"]], hi[nd["name"]] = a.abs().sqrt(), h.abs().sqrt()
    return {"sums": np.array(sums), "verdicts": None, "status": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return _exact_batch(case, seed)
    inp = _inputs(case, seed)
    if kind == "train":
        return _exact_train(case, inp, seed)
    if kind == "chain":
        s = float((2 * inp["x"].double() + 1 + inp["y"].double()).sum())
        return {"verdicts": None, "s": s, "shadow": s}
    if kind == "filter":
        # which items are kept is decided on the float32 chain (each step rounded), their values
        # and the reductions are those of the chain in 64 bits
        f = lambda t: t.float().double()
        x, y = inp["x"].double(), inp["y"].double()
        u = f(f(x * W.CFG2_A) + W.CFG2_B)
        kept = f(f(torch.exp(-f(u * u))) * y) > float(np.float32(W.CFG2_T))
        k = (torch.exp(-(x * W.CFG2_A + W.CFG2_B) ** 2) * y)[kept]
        s = float(k.sum())
        m = float(k.max()) if k.numel() else -math.inf
        k = torch.cat([k, k.new_zeros(case["n"] - k.numel())])
        return {"verdicts": None, "k": k, "s": s, "shadow": s, "m": m, "c": None}
    if kind == "product":
        return {"verdicts": None, "C": inp["A"].double() @ inp["B"].double()}
    if kind == "sort":
        return {"verdicts": None, "r": inp["a"].double().sort().values} if case["dtype"] == "f32" else None
    if kind == "transpose":
        return {"verdicts": None, "T": inp["M"].double().t().contiguous()}
    if kind == "matvec":
        M, v = inp["M"].double(), inp["v"].double()
        y = M @ v
        return {"y": y, "z": y @ M}
    if kind == "det":
        lu, piv = torch.linalg.lu_factor(inp["A"].double().cpu())
        mant, expo = 1.0, 0
        for d in lu.diagonal().tolist():
            mant, e = math.frexp(mant * d)
            expo += e
        return {"verdicts": None, "sign": None, "mant": abs(mant), "expo": None}
    return None
