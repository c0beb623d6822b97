"""The calls whose time this framework answers for, and the ranges around them.

``listed()`` names them, ``draw(rng)`` makes another of the same ranges,
``prepare`` builds what a user's program has in hand before the call (the
graph handle, the signal on the device, the weights), ``run`` is one pass
through the public entry points, ``work`` the bytes and operations of a pass
that no implementation can avoid, and ``exact`` the truncated sum of the
propagation in binary64.

A case's "kind" is one of
  propagate  agp.propagate of C columns ("dtype" f32 or f64, "split" for the
             literal x+/x- treatment of signed signals)
  noalloc    agp.propagate_noalloc (callers that cannot allocate)
  cluster    agp.propagate of C seeds and the conductance sweep of every
             column (agp.sweep with the order for one, agp.sweep_batch for more)
  serve      C queries submitted to an agp.Server and polled to the end
Its "graph" is chung_lu (degree "deg", exponent "gamma", optional self-loops)
or rmat ("deg" generated edges per node), each symmetrised, or rmat_directed
(out-arcs as generated).  "model" is ppr, hkpr, katz, tp or target
(single-target PPR); "signal" onehot, normal or uniform.
"""
import math
import time

import numpy as np
import torch

from paper_2106_03058_amd import agp, inputs

DEV = "cuda:0"
RMAT = (0.57, 0.19, 0.19)
# exponents (a, b) of D^-a A D^-b of every model; the GNN signals use 1/2, 1/2
EXPONENTS = {"ppr": (0.0, 1.0), "hkpr": (0.0, 1.0), "tp": (0.0, 1.0), "katz": (0.0, 0.0), "target": (1.0, 0.0)}


def _case(name=None, **kw):
    case = {"kind": "propagate", "graph": "chung_lu", "n": 10000, "deg": 10.0, "gamma": 2.5, "loops": False,
            "model": "ppr", "param": 0.2, "L": 20, "eps": 1e-6, "C": 1, "signal": "onehot", "dtype": "f32",
            "split": False}
    case.update(kw)
    if name is not None:
        case["name"] = name
    return case


def listed():
    return [
        # one proximity query at a time on a small graph: the smallest call a
        # program makes, and it makes many of them
        _case("ppr_query", n=10000, C=1),
        # the same graph in binary64, where the estimate feeds further analysis
        _case("ppr_f64", n=10000, C=3, dtype="f64"),
        # a tight serving loop that must not allocate, a handful of queries a call
        _case("ppr_noalloc", kind="noalloc", n=30011, C=9, L=15, eps=1e-5),
        # similarity to a few targets in a directed (follower-style) graph
        _case("target_directed", graph="rmat_directed", n=1 << 17, deg=16.0, model="target", C=33, eps=1e-6),
        # a block of Katz queries on a social graph
        _case("katz_block", graph="rmat", n=1 << 20, deg=16.0, model="katz", param=0.85, L=30, eps=1e-7, C=64),
        # ten-step transition probabilities from many sources, dense levels
        _case("tp_block", graph="rmat", n=1 << 22, deg=16.0, model="tp", L=10, eps=1e-7, C=64),
        # heat-kernel smoothing of a GNN's whole feature matrix
        _case("gnn_hkpr", n=2400000, deg=50.0, loops=True, model="hkpr", param=5.0, L=10, eps=1e-7, C=128,
              signal="normal"),
        # PPR smoothing of features on a large sparse graph, coarse threshold
        _case("gnn_ppr", n=8000000, deg=14.5, gamma=2.2, loops=True, model="ppr", param=0.1, L=10, eps=1.4e-7, C=32,
              signal="uniform"),
        # signed features propagated as two parts, an odd number of them
        _case("gnn_split", n=200003, deg=30.0, loops=True, model="hkpr", param=5.0, L=10, eps=1e-6, C=11,
              signal="normal", split=True),
        # the cluster around one seed: estimate and sweep, interactive use
        _case("cluster_seed", kind="cluster", n=400009, deg=40.0, gamma=2.3, model="hkpr", param=5.0, L=20, eps=1e-6,
              C=1),
        # the clusters around many seeds at once
        _case("cluster_block", kind="cluster", n=600011, deg=76.0, gamma=2.3, model="hkpr", param=5.0, L=20, eps=1e-6,
              C=64),
        # a burst of mixed queries (PPR, Katz, transition probabilities) to the server
        _case("serve_burst", kind="serve", graph="rmat", n=1 << 18, deg=32.0, model="mix", eps=1e-6, C=48),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "noalloc", "directed", "block", "gnn", "split", "cluster", "serve"])
    n = _logint(rng, 5000, 40000)
    if kind == "small":
        return _case(n=n, deg=rng.uniform(6.0, 30.0), C=_logint(rng, 1, 12), L=rng.randint(8, 25),
                     eps=10.0 ** rng.uniform(-6.5, -4.5), dtype=rng.choice(["f32", "f64"]),
                     model=rng.choice(["ppr", "tp"]))
    if kind == "noalloc":
        return _case(kind="noalloc", n=n, deg=rng.uniform(6.0, 20.0), C=_logint(rng, 1, 40), L=rng.randint(5, 20),
                     eps=10.0 ** rng.uniform(-6.0, -4.5))
    if kind == "directed":
        return _case(graph="rmat_directed", n=1 << rng.randint(14, 19), deg=16.0, model=rng.choice(["ppr", "target"]),
                     C=_logint(rng, 4, 70), eps=10.0 ** rng.uniform(-7.0, -5.0))
    if kind == "block":
        model = rng.choice(["katz", "tp"])
        return _case(graph="rmat", n=1 << rng.randint(16, 21), deg=16.0, model=model, C=_logint(rng, 5, 64),
                     L=30 if model == "katz" else rng.randint(4, 10), param=0.85, eps=10.0 ** rng.uniform(-7.0, -5.5))
    if kind == "gnn":
        n, C = _logint(rng, 60000, 2000000), _logint(rng, 7, 128)
        model = rng.choice(["hkpr", "ppr"])
        return _case(n=n, deg=rng.uniform(10.0, 50.0), gamma=rng.uniform(2.2, 2.5), loops=True, model=model,
                     param=5.0 if model == "hkpr" else 0.1, L=10, eps=rng.uniform(0.2, 1.1) / n, C=C,
                     signal=rng.choice(["normal", "uniform"]))
    if kind == "split":
        return _case(n=_logint(rng, 20000, 400000), deg=rng.uniform(10.0, 50.0), loops=True, model="hkpr", param=5.0,
                     L=rng.randint(6, 12), eps=10.0 ** rng.uniform(-6.5, -5.5), C=_logint(rng, 3, 24),
                     signal="normal", split=True)
    if kind == "cluster":
        return _case(kind="cluster", n=_logint(rng, 30000, 600000), deg=rng.uniform(20.0, 76.0), gamma=2.3,
                     model="hkpr", param=5.0, L=20, eps=10.0 ** rng.uniform(-6.5, -5.5),
                     C=rng.choice([1, _logint(rng, 2, 64)]))
    return _case(kind="serve", graph="rmat", n=1 << rng.randint(15, 18), deg=32.0, model="mix",
                 eps=10.0 ** rng.uniform(-6.0, -5.0), C=rng.randint(16, 60))


# ------------------------------------------------------------------ inputs

def _csr(case, seed):
    """The case's graph as device CSR tensors (int64 row_ptr, int32 col)."""
    n = case["n"]
    if case["graph"] == "chung_lu":
        _, rp, col = inputs.chung_lu_device(n, case["deg"], case["gamma"], seed)
        if case["loops"]:
            rp, col = inputs.add_self_loops_device(n, rp, col)
        return rp, col
    scale = n.bit_length() - 1
    if case["graph"] == "rmat":
        _, rp, col = inputs.rmat_device(scale, int(case["deg"]), *RMAT, seed)
        return rp, col
    # directed: one R-MAT arc list, tails and heads as generated
    gen = torch.Generator(device=DEV).manual_seed(seed)
    m = int(n * case["deg"])
    s = torch.zeros(m, dtype=torch.int64, device=DEV)
    d = torch.zeros(m, dtype=torch.int64, device=DEV)
    a, b, c = RMAT
    for _ in range(scale):
        u = torch.rand(m, generator=gen, device=DEV)
        s = s * 2 + (u >= a + b)
        d = d * 2 + (((u >= a) & (u < a + b)) | (u >= a + b + c))
    key = torch.unique((s * n + d)[s != d])
    rows = torch.div(key, n, rounding_mode="floor")
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return rp, (key - rows * n).to(torch.int32)


def _sources(rp, k, seed):
    """k nodes drawn uniformly over the nodes that have arcs."""
    cand = torch.nonzero(rp[1:] > rp[:-1]).flatten()
    gen = torch.Generator().manual_seed(seed + 1)
    return cand[torch.randint(cand.numel(), (k,), generator=gen).to(DEV)]


def _signal(case, rp, seed):
    n, C = case["n"], case["C"]
    dtype = torch.float64 if case["dtype"] == "f64" else torch.float32
    if case["signal"] == "onehot":
        x = torch.zeros((n, C), dtype=dtype, device=DEV)
        x[_sources(rp, C, seed), torch.arange(C, device=DEV)] = 1.0
        return x
    gen = torch.Generator(device=DEV).manual_seed(seed + 2)
    if case["signal"] == "normal":
        return torch.randn((n, C), generator=gen, device=DEV, dtype=dtype)
    return torch.rand((n, C), generator=gen, device=DEV, dtype=dtype).mul_(2.0).sub_(1.0)


def _katz_beta(rp, col, scale):
    """scale over an estimate of the largest adjacency eigenvalue, the exact
    integer moment ratio d^T A d / d^T d of the degrees (at most lambda_1)."""
    d = rp[1:] - rp[:-1]
    tails = torch.repeat_interleave(d, d)
    return scale * float((d * d).sum().item()) / float((tails * d[col.long()]).sum().item())


def _weights(case, beta=None):
    L, p = case["L"], case["param"]
    if case["model"] in ("ppr", "target"):
        return inputs.weights_ppr(p, L)
    if case["model"] == "hkpr":
        return inputs.weights_hkpr(p, L)
    if case["model"] == "katz":
        return inputs.weights_katz(beta, L, 0.85)
    return inputs.weights_tp(L)


def _exponents(case):
    return EXPONENTS[case["model"]] if case["signal"] == "onehot" else (0.5, 0.5)


def _queries(case, rp, beta, seed):
    """The burst: a third each of PPR, Katz and transition probabilities."""
    rng = np.random.default_rng(seed)
    src = _sources(rp, case["C"], seed).tolist()
    qs = []
    for i, s in enumerate(src):
        L = int(rng.integers(10, 31))
        eps = case["eps"] * float(rng.choice([1.0, 3.0, 10.0]))
        if i % 3 == 0:
            a, b, w = 0.0, 1.0, inputs.weights_ppr(float(rng.uniform(0.1, 0.3)), L)
        elif i % 3 == 1:
            a, b, w = 0.0, 0.0, inputs.weights_katz(beta, L, 0.85)
        else:
            a, b, w = 0.0, 1.0, inputs.weights_tp(L)
        qs.append((s, a, b, w, eps, seed, i))
    return qs


def prepare(case, seed):
    rp, col = _csr(case, seed)
    directed = case["graph"] == "rmat_directed"
    state = {"case": case, "seed": seed,
             "graph": agp.Graph(rp, col, directed=directed, reverse=directed and case["model"] == "target")}
    beta = _katz_beta(rp, col, 0.85) if case["model"] in ("katz", "mix") else None
    if case["kind"] == "serve":
        state["queries"] = _queries(case, rp, beta, seed)
        state["outs"] = [torch.empty(case["n"], dtype=torch.float32, device=DEV) for _ in range(case["C"])]
        state["server"] = agp.Server(state["graph"], max_slots=32, queue_capacity=256, memory_bytes=4 << 30)
        return state
    state["x"] = _signal(case, rp, seed)
    state["w"] = _weights(case, beta)
    if case["kind"] == "noalloc":
        state["out"] = torch.empty_like(state["x"])
        # the entry point needs the graph's degree powers: one ordinary call makes them
        agp.propagate(state["graph"], *_exponents(case), state["w"], state["x"][:, :1].contiguous(), 1e-2, seed)
    return state


def run(state):
    case, g, seed = state["case"], state["graph"], state["seed"]
    if case["kind"] == "serve":
        srv = state["server"]
        todo = [srv.submit(*q, out) for q, out in zip(state["queries"], state["outs"])]
        while todo:
            todo = [t for t in todo if srv.poll(t) is None]
            if todo:
                time.sleep(5e-5)
        return state["outs"]
    a, b = _exponents(case)
    if case["kind"] == "noalloc":
        return agp.propagate_noalloc(g, a, b, state["w"], state["x"], case["eps"], seed, out=state["out"])
    pi, _ = agp.propagate(g, a, b, state["w"], state["x"], case["eps"], seed, split_signs=case["split"])
    if case["kind"] != "cluster":
        return pi
    if case["C"] == 1:
        size, phi, order = agp.sweep(g, pi[:, 0])
        return {"pi": pi, "size": size, "phi": phi, "order": order}
    size, phi = agp.sweep_batch(g, pi)
    return {"pi": pi, "size": size, "phi": phi}


# -------------------------------------------------------------------- work

def _arcs(case):
    both = 1 if case["graph"] == "rmat_directed" else (1 if case["graph"] == "chung_lu" else 2)
    return case["n"] * case["deg"] * both + (case["n"] if case["loops"] else 0)


def work(case):
    """Every input read once and every output written once (the signal and
    the estimate of C columns, the adjacency lists as far as the call reaches
    them), and a multiply and an add per edge push: a level pushes along at
    most every arc of a column and, in expectation, 1 / eps times."""
    n, C, L = case["n"], case["C"], 20 if case["kind"] == "serve" else case["L"]
    arcs = _arcs(case)
    size = 8 if case["dtype"] == "f64" else 4
    pushes = C * L * min(arcs, 1.0 / case["eps"])
    dense = n * C * size
    if case["kind"] == "serve":
        nbytes = dense  # single-source queries: only the estimates are dense
    else:
        nbytes = 2 * dense
    nbytes += min(4 * arcs, 4 * pushes) + min(12 * n, 12 * pushes)
    if case["kind"] == "cluster":
        nbytes += (4 * n if C == 1 else 16 * C) + 4 * arcs
    return {"bytes": int(nbytes), "flops": int(2 * pushes)}


# ------------------------------------------------------------------- exact

def _horner(n, rows, cols, fa, fb, w, x):
    """sum_i w_i (D^-a A D^-b)^i x column block by column block; w is (L + 1)
    or (L + 1) x C."""
    y = x * w[-1]
    for wi in reversed(w[:-1]):
        z = torch.zeros_like(y)
        z.index_add_(0, cols, (y * fb)[rows])
        y = z * fa + x * wi
    return y


def exact(case, seed):
    """The truncated sum of Eq. 1 in binary64 (arcs pushed from tail to head;
    against the arcs for a single target).  None beyond a few seconds' work,
    and for feature matrices, whose estimates are mostly sampling noise at
    their thresholds (eps ||x||_1 is a fair part of an entry)."""
    C, L = case["C"], 30 if case["kind"] == "serve" else case["L"]
    if case["signal"] != "onehot" or _arcs(case) * C * L > 4e9:
        return None
    n = case["n"]
    rp, col = _csr(case, seed)
    d = rp[1:] - rp[:-1]
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), d)
    cols = col.long()
    beta = _katz_beta(rp, col, 0.85) if case["model"] in ("katz", "mix") else None
    df = d.clamp(min=1).double()[:, None]

    def factors(a, b):
        return df ** -a, df ** -b

    if case["kind"] == "serve":
        res = []
        for s, a, b, w, _, _, _ in _queries(case, rp, beta, seed):
            x = torch.zeros((n, 1), dtype=torch.float64, device=DEV)
            x[s] = 1.0
            res.append(_horner(n, rows, cols, *factors(a, b), w, x)[:, 0])
        return res
    if case["graph"] == "rmat_directed" and case["model"] == "target":
        rows, cols = cols, rows
    w, ab = _weights(case, beta), factors(*_exponents(case))
    x = _signal(case, rp, seed).double()
    pi = torch.cat([_horner(n, rows, cols, *ab, w, x[:, c:c + 4]) for c in range(0, C, 4)], 1)
    if case["kind"] != "cluster":
        return pi
    out = {"pi": pi, "size": None, "phi": None}
    if C == 1:
        out["order"] = None
    return out
