"""Workloads by which the speed of this framework is measured.

Each case is one call, or one short sequence of calls, that a graph-network
program makes through the package's public entry points (``Plan``,
``Plan.spmm``, ``Plan.gcn_layer``, ``linear``), on graphs of the three kinds
the framework is built for: Erdos-Renyi, power-law (Chung-Lu) and skewed-hub
graphs, from a few thousand rows to 2.4 million.

Operations:

* ``spmm``        aggregation Y = A X over a plan built once (training and
                  inference aggregate many times over one graph; under the
                  symmetric normalisation the backward product is the same call)
* ``fresh_spmm``  plan and aggregation(s) on a graph seen for the first time
* ``layer``       one GCNConv forward act(A (X W)) over a plan built once
* ``fresh_layer`` plan and one GCNConv forward (a sampled subgraph per step)
* ``gcn2``        a two-layer model, logits out
* ``linear``      the feature transformation X W alone

All data is float32 with int32 indices, the types the framework takes.
"""
import math

import torch

import paper_2308_11825_amd as agcn

DEVICE = "cuda:0"


def listed():
    return [
        # A small graph's aggregation: launch latency and host time count.
        dict(name="tiny_spmm", op="spmm", graph="er", n=4096, mean=8, F=16),
        # A sampled subgraph: a new graph at every step, used for one layer.
        dict(name="subgraph_layer", op="fresh_layer", graph="powerlaw", n=12000, mean=10,
             alpha=2.2, cap=600, fin=128, fout=64, act="relu"),
        # A citation-size graph, one aggregation at a narrow width.
        dict(name="medium_spmm", op="spmm", graph="powerlaw", n=170000, mean=14, alpha=2.1,
             cap=5000, F=32),
        # Two-layer model on the same graph: 128 features, 256 hidden, 40 classes.
        dict(name="medium_gcn2", op="gcn2", graph="powerlaw", n=170000, mean=14, alpha=2.1,
             cap=5000, fin=128, hidden=256, fout=40),
        # The benchmark's step: a plan, then the aggregation at five widths.
        dict(name="sweep_step", op="fresh_spmm", graph="powerlaw", n=230000, mean=50, alpha=2.0,
             cap=3391, F="16,32,64,128,256"),
        # Aggregation of class scores: an odd width, rows not 16-byte aligned.
        dict(name="sweep_spmm_odd", op="spmm", graph="powerlaw", n=230000, mean=50, alpha=2.0,
             cap=3391, F=41),
        # A hidden layer of a model on the benchmark's graph.
        dict(name="sweep_layer", op="layer", graph="powerlaw", n=230000, mean=50, alpha=2.0,
             cap=3391, fin=128, fout=128, act="relu"),
        # First layers' transformation: wide raw features, many rows.
        dict(name="linear_wide", op="linear", n=230000, fin=602, fout=256),
        # The same on a small graph with bag-of-words features.
        dict(name="linear_small", op="linear", n=3000, fin=1000, fout=16),
        # Aggregation with ReLU on a million-node graph at an unrounded width.
        dict(name="million_spmm", op="spmm", graph="powerlaw", n=1000000, mean=20, alpha=2.2,
             cap=4000, F=100, act="relu"),
        # The largest power-law graph, features far larger than any cache.
        dict(name="large_spmm", op="spmm", graph="powerlaw", n=2400000, mean=50, alpha=2.3,
             cap=10954, F=128),
        # A thousand very long rows hold nearly all nonzeros; plan included.
        dict(name="hubs_step", op="fresh_spmm", graph="hubs", n=1000000, hubs=1000, lo=20000,
             hi=200000, F="64"),
    ]


#: No drawn case has more (nonzeros x feature columns) than the largest listed one.
MOST_NNZ = 120_000_000
MOST_NNZ_F = 120_000_000 * 128


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, hi=256):
    """Feature widths: powers of two, other multiples of four, odd ones."""
    kind = rng.random()
    if kind < 0.4:
        return min(hi, rng.choice([16, 32, 64, 128, 256]))
    if kind < 0.7:
        return 4 * rng.randint(1, hi // 4)
    return _log(rng, 3, hi)


def draw(rng):
    op = rng.choice(["spmm", "spmm", "spmm", "fresh_spmm", "layer", "fresh_layer", "gcn2", "linear"])
    if op == "linear":
        n = _log(rng, 2000, 2_400_000)
        fin = _log(rng, 16, 1500)
        while n * fin > 400_000_000:
            fin = max(16, fin // 2)
        return dict(op=op, n=n, fin=fin, fout=_width(rng))
    most_n = 60_000 if op == "fresh_layer" else 2_400_000
    n = _log(rng, 3000, most_n)
    kind = rng.choice(["er", "powerlaw", "powerlaw", "powerlaw", "hubs"])
    c = dict(op=op, graph=kind, n=n)
    if kind == "hubs":
        c["hubs"] = rng.randint(70, max(80, min(1200, n // 100)))
        c["hi"] = max(600, n // rng.randint(5, 40))
        c["lo"] = max(520, c["hi"] // 10)
        nnz = n * 4.5 + c["hubs"] * (c["lo"] + c["hi"]) / 2
        if nnz > MOST_NNZ:
            c["hubs"] = max(70, int(c["hubs"] * MOST_NNZ / nnz / 1.1))
            nnz = n * 4.5 + c["hubs"] * (c["lo"] + c["hi"]) / 2
    else:
        c["mean"] = _log(rng, 4, 60)
        if kind == "powerlaw":
            c["alpha"] = round(rng.uniform(2.0, 2.5), 2)
            c["cap"] = max(200, int(math.sqrt(n * c["mean"]) * rng.choice([0.5, 1.0, 2.0])))
            c["cap"] = min(c["cap"], n // 4)
        nnz = n * (c["mean"] + 1.0)
    if op in ("spmm", "fresh_spmm"):
        widths = [_width(rng)] if op == "spmm" or rng.random() < 0.5 else [16, _width(rng)]
        while sum(widths) * nnz > MOST_NNZ_F:
            widths = [max(4, w // 2) for w in widths]
        c["F"] = widths[0] if op == "spmm" else ",".join(str(w) for w in widths)
        if op == "spmm":
            c["act"] = rng.choice(["none", "relu"])
    else:
        c["fin"], c["fout"] = _width(rng), _width(rng)
        if op == "gcn2":
            c["hidden"] = rng.choice([16, 64, 100, 128, 256])
        else:
            c["act"] = rng.choice(["none", "relu"])
        while (c["fin"] + c["fout"] + c.get("hidden", 0)) * nnz > MOST_NNZ_F:
            c["fin"], c["fout"] = max(8, c["fin"] // 2), max(8, c["fout"] // 2)
            if "hidden" in c:
                c["hidden"] = max(16, c["hidden"] // 2)
    # Columns of a row in arbitrary order, as an edge list gives them.
    if rng.random() < 0.15:
        c["shuffled"] = True
    return c


# --- inputs ---------------------------------------------------------------------


def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _csr(n, keys, gen, shuffled):
    """CSR of the distinct sorted keys row * n + column, values 1 / sqrt(d_i d_j)."""
    rows = torch.div(keys, n, rounding_mode="floor")
    cols = keys - rows * n
    deg = torch.bincount(rows, minlength=n)
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEVICE)
    torch.cumsum(deg, 0, out=rowptr[1:])
    if shuffled:
        salt = torch.randint(0, 1 << 20, (keys.numel(),), generator=gen, device=DEVICE)
        cols = cols[torch.argsort((rows << 20) | salt, stable=True)]
    d = deg.clamp(min=1).double()
    vals = (1.0 / torch.sqrt(d[rows] * d[cols])).float()
    return rowptr.int(), cols.int(), vals


def _graph(case, gen):
    n = case["n"]
    kind = case["graph"]
    diag = torch.arange(n, dtype=torch.int64, device=DEVICE) * (n + 1)
    if kind == "er":
        m = int(n * case["mean"])
        keys = torch.randint(0, n * n, (m,), generator=gen, device=DEVICE)
        keys = torch.unique(torch.cat([keys, diag]))
    elif kind == "powerlaw":
        # Chung-Lu: endpoints drawn in proportion to Zipf(alpha) expected degrees.
        u = torch.rand(n, generator=gen, device=DEVICE, dtype=torch.float64)
        w = torch.floor(u.clamp(min=1e-12).pow(-1.0 / (case["alpha"] - 1.0)))
        for _ in range(3):
            w = (w * (case["mean"] / w.mean())).clamp(1.0, float(case["cap"]))
        cdf = torch.cumsum((w * (1 << 16)).long(), 0)  # whole numbers: the same every time
        m = int(round(n * case["mean"] / 2))
        ends = torch.searchsorted(cdf, torch.randint(0, int(cdf[-1]), (2 * m,), generator=gen,
                                                     device=DEVICE), right=True)
        lo, hi = torch.minimum(ends[:m], ends[m:]), torch.maximum(ends[:m], ends[m:])
        und = torch.unique((lo * n + hi)[lo != hi])
        lo = torch.div(und, n, rounding_mode="floor")
        hi = und - lo * n
        keys = torch.sort(torch.cat([und, hi * n + lo, diag])).values
    else:
        # Rows of degree 1 to 8, and `hubs` rows of degree lo to hi.
        hub = torch.randperm(n, generator=gen, device=DEVICE)[: case["hubs"]]
        deg = torch.randint(1, 9, (n,), generator=gen, device=DEVICE)
        deg[hub] = torch.randint(case["lo"], case["hi"] + 1, (hub.numel(),), generator=gen,
                                 device=DEVICE)
        rows = torch.repeat_interleave(torch.arange(n, device=DEVICE), deg)
        cols = torch.randint(0, n, (rows.numel(),), generator=gen, device=DEVICE)
        keys = torch.unique(rows * n + cols)
    return _csr(n, keys, gen, case.get("shuffled", False))


def _features(n, f, gen):
    return torch.randn((n, f), generator=gen, device=DEVICE)


def _weights(fin, fout, gen):
    lim = math.sqrt(6.0 / (fin + fout))
    return (torch.rand((fin, fout), generator=gen, device=DEVICE) * 2 - 1) * lim


def _widths(case):
    return [int(f) for f in str(case["F"]).split(",")]


def _inputs(case, seed):
    gen = _generator(seed)
    s = {}
    if case["op"] != "linear":
        s["csr"] = _graph(case, gen)
    n = case["n"]
    if "F" in case:
        s["X"] = [_features(n, f, gen) for f in _widths(case)]
    else:
        s["X"] = _features(n, case["fin"], gen)
        if case["op"] == "gcn2":
            s["W1"] = _weights(case["fin"], case["hidden"], gen)
            s["W2"] = _weights(case["hidden"], case["fout"], gen)
        else:
            s["W"] = _weights(case["fin"], case["fout"], gen)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    if case["op"] in ("spmm", "layer", "gcn2"):
        s["plan"] = agcn.Plan(*s["csr"], n_cols=case["n"])
        del s["csr"]  # the plan holds its own copy
    return s


def run(s):
    case = s["case"]
    op, act = case["op"], case.get("act", "none")
    if op == "linear":
        return agcn.linear(s["X"], s["W"])
    if op == "spmm":
        return s["plan"].spmm(s["X"][0], act=act)
    if op == "layer":
        return s["plan"].gcn_layer(s["X"], s["W"], act=act)
    if op == "gcn2":
        h = s["plan"].gcn_layer(s["X"], s["W1"], act="relu")
        return s["plan"].gcn_layer(h, s["W2"], act="none")
    plan = agcn.Plan(*s["csr"], n_cols=case["n"])
    if op == "fresh_layer":
        return plan.gcn_layer(s["X"], s["W"], act=act)
    return [plan.spmm(x) for x in s["X"]]


# --- the work a pass cannot do without, and its results in 64 bits -----------------


def _nnz(case):
    n = case["n"]
    if case["graph"] == "hubs":
        return n * 4.5 + case["hubs"] * (case["lo"] + case["hi"]) / 2
    return n * (case["mean"] + 1.0)


def work(case):
    n = case["n"]
    if case["op"] == "linear":
        fin, fout = case["fin"], case["fout"]
        return {"bytes": 4 * (n * fin + fin * fout + n * fout), "flops": 2 * n * fin * fout}
    nnz = _nnz(case)
    b, f = 8 * nnz + 4 * n, 0
    if "F" in case:
        for w in _widths(case):
            b += 8 * n * w
            f += 2 * nnz * w
    else:
        chain = [case["fin"]] + ([case["hidden"]] if "hidden" in case else []) + [case["fout"]]
        b += 4 * n * (chain[0] + chain[-1])
        for i, o in zip(chain, chain[1:]):
            b += 4 * i * o
            # A (X W) and (A X) W are the same layer: the cheaper aggregation.
            f += 2 * n * i * o + 2 * nnz * min(i, o)
    return {"bytes": b, "flops": f}


def tolerance(case):
    # Against 64 bits the aggregations measure 4e-8 to 8e-8 (other orders of a
    # long row's sum reach a few times that), the transformations 2e-7 to
    # 6e-7 with 100 to 1000 terms per element: four times those.
    rel = 5e-7 if case["op"] in ("spmm", "fresh_spmm") else 2.5e-6
    return {"rel": rel, "max": 100 * rel}


def _spmm64(csr, X):
    rowptr, cols, vals = csr
    n, f = rowptr.numel() - 1, X.shape[1]
    X = X.double()
    Y = torch.zeros((n, f), dtype=torch.float64, device=DEVICE)
    deg = (rowptr[1:] - rowptr[:-1]).long()
    rows = torch.repeat_interleave(torch.arange(n, device=DEVICE), deg)
    step = max(1, (1 << 29) // f)
    for a in range(0, cols.numel(), step):
        part = X[cols[a:a + step].long()]
        part *= vals[a:a + step].double()[:, None]
        Y.index_add_(0, rows[a:a + step], part)
    return Y


def exact(case, seed):
    s = _inputs(case, seed)
    op, act = case["op"], case.get("act", "none")
    if op == "linear":
        return s["X"].double() @ s["W"].double()
    csr = s["csr"]
    if "F" in case:
        ys = [_spmm64(csr, x) for x in s["X"]]
        if op == "spmm":
            return ys[0].clamp(min=0) if act == "relu" else ys[0]
        return ys
    if op == "gcn2":
        h = _spmm64(csr, s["X"].double() @ s["W1"].double()).clamp(min=0)
        return _spmm64(csr, h @ s["W2"].double())
    y = _spmm64(csr, s["X"].double() @ s["W"].double())
    return y.clamp(min=0) if act == "relu" else y
