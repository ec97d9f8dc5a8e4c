"""Performance cases of the triangle-counting library, as its users call it.

A case is one call (or one queue of calls) through the package's public entry
points on a synthetic graph drawn on the GPU from a seed: R-MAT (scale-free,
the benchmark's family), Chung-Lu power law (the batch's family), random
geometric (mesh-like), uniform with repeats, and Erdos-Renyi without repeats.
Sizes are those of ``bench.py`` and the tests, or ragged ones between them.
"""
from __future__ import annotations

import json
import math
import os

import numpy as np
import torch

import paper_1804_06926_amd as tc

DEVICE = "cuda:0"
GAMMA = 2.1                      # Chung-Lu exponent of the benchmark's batch
RMAT_ABC = (0.57, 0.19, 0.19)    # d = 0.05
SELECT = {"heuristic": tc.SELECT_HEURISTIC, "learned": tc.SELECT_LEARNED}
WEIGHTS = os.path.join(os.path.dirname(tc.__file__), "selector_weights.json")


def listed():
    return [
        # one request of a service that counts a small graph and waits for the answer: pure latency
        dict(name="er_4096", call="count", graph="er", n=4096, pairs=32768, per_vertex=True, select="heuristic"),
        # a stream of small graphs (ego networks, molecules of a data set) queued without waiting in between
        dict(name="queue_chung_lu", call="queue", graph="chung_lu", graphs=64, lo=1000, hi=100000,
             select="heuristic"),
        # per-vertex counts inside a loop that may not allocate; largest kind of graph the fixed scratch takes
        dict(name="noalloc_rmat_16", call="noalloc", graph="rmat", scale=16, pairs=1 << 20, per_vertex=True,
             select="heuristic"),
        # the usual scale-free graph of a few ten million edges, count only
        dict(name="rmat_20", call="count", graph="rmat", scale=20, pairs=16 << 20, per_vertex=False,
             select="heuristic"),
        # the headline: a quarter of a billion pairs
        dict(name="rmat_24", call="count", graph="rmat", scale=24, pairs=16 << 24, per_vertex=False,
             select="heuristic"),
        # a mesh-like graph (short, even neighbour lists), strategy picked by the trained selector
        dict(name="rgg_23", call="count", graph="rgg", n=1 << 23, degree=32.0, per_vertex=False, select="learned"),
        # raw log data: ragged sizes, repeats and loops, hardly any triangles; counts wanted per vertex
        dict(name="uniform_ragged", call="count", graph="uniform", n=1000003, pairs=10000019, per_vertex=True,
             select="heuristic"),
        # many graphs of very different sizes in one captured call
        dict(name="batch_chung_lu", call="batch", graph="chung_lu", graphs=1024, lo=1000, hi=1000000,
             select="heuristic"),
        # clustering coefficients of a social-network-like graph
        dict(name="clustering_rmat_18", call="clustering", graph="rmat", scale=18, pairs=16 << 18,
             select="heuristic"),
        # triangles per edge, the input of k-truss, on a ragged power-law graph without repeats
        dict(name="support_chung_lu", call="support", graph="chung_lu", distinct=True, n=777777, pairs=6000001,
             select="heuristic"),
        # the degree-ordered CSR alone, for a user's own kernels
        dict(name="csr_rmat_22", call="csr", graph="rmat", distinct=True, scale=22, pairs=50000017),
        # one evaluation of the selector network while it is trained: logits, loss and gradient
        dict(name="selector_691", call="selector", batch=691),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: any call, family and option, sizes log-uniform, mostly odd."""
    call = rng.choice(["count", "count", "count", "count", "queue", "noalloc", "batch", "clustering", "support",
                       "edge_counts", "csr", "selector"])
    if call == "selector":
        return dict(call=call, batch=_log_uniform(rng, 16, 65536))
    select = rng.choice(["heuristic", "heuristic", "learned"])
    if call == "queue":
        return dict(call=call, graph="chung_lu", graphs=rng.randint(8, 96), lo=_log_uniform(rng, 100, 2000),
                    hi=_log_uniform(rng, 5000, 200000), select=select)
    if call == "batch":
        return dict(call=call, graph="chung_lu", graphs=_log_uniform(rng, 16, 1024), lo=_log_uniform(rng, 200, 5000),
                    hi=_log_uniform(rng, 20000, 1000000), select=select)
    if call == "noalloc":
        case = dict(call=call, select=select, per_vertex=rng.random() < 0.5,
                    **_draw_graph(rng, 500, 1 << 20, ["er", "rmat", "chung_lu", "uniform"]))
    elif call == "clustering":
        case = dict(call=call, select=select,
                    **_draw_graph(rng, 2000, 16 << 18, ["rmat", "rgg", "chung_lu", "uniform"]))
    elif call != "count":   # outputs per edge: their number is fixed by a simple graph of so many pairs
        case = dict(call=call, select=select, distinct=True,
                    **_draw_graph(rng, 8000, (16 << 18) if call == "support" else (1 << 26),
                                  ["er", "rmat", "chung_lu", "uniform"]))
    else:
        case = dict(call=call, select=select,
                    **_draw_graph(rng, 1000, 1 << 27, ["er", "rmat", "rmat", "rgg", "chung_lu", "uniform"]))
    if call == "count":
        case["per_vertex"] = rng.random() < 0.3
    return case


def _draw_graph(rng, lo, hi, families):
    family = rng.choice(families)
    if family == "er":
        pairs = _log_uniform(rng, lo, min(hi, 1 << 20))
        return dict(graph=family, n=max(pairs // rng.randint(4, 16), 64), pairs=pairs)
    pairs = _log_uniform(rng, lo, hi)
    if family == "rmat":   # 8 to 32 pairs per vertex
        return dict(graph=family, scale=max(6, int(math.log2(pairs / rng.uniform(8, 32)))), pairs=pairs)
    if family == "rgg":
        degree = rng.choice([16.0, 32.0])
        return dict(graph=family, n=max(64, int(2 * pairs / degree)), degree=degree)
    return dict(graph=family, n=max(16, int(pairs / rng.uniform(6, 16))), pairs=pairs)


# ---------------------------------------------------------------- inputs
def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _rand(size, gen, dtype=torch.float32):
    return torch.rand(size, generator=gen, device=DEVICE, dtype=dtype)


def _shuffled(pairs, gen):
    """The pairs in random order, each in a random direction."""
    pairs = pairs[torch.randperm(pairs.shape[0], generator=gen, device=DEVICE)]
    flip = _rand(pairs.shape[0], gen) < 0.5
    return torch.where(flip[:, None], pairs.flip(1), pairs).to(torch.int32).contiguous()


def _rmat(scale, pairs, gen):
    """Raw R-MAT draws (repeats and loops included) under a random vertex permutation, random direction."""
    a, b, c = RMAT_ABC
    perm = torch.randperm(1 << scale, generator=gen, device=DEVICE).to(torch.int32)
    out = torch.empty((pairs, 2), dtype=torch.int32, device=DEVICE)
    for s in range(0, pairs, 1 << 26):
        k = min(1 << 26, pairs - s)
        u = torch.zeros(k, dtype=torch.int32, device=DEVICE)
        v = torch.zeros(k, dtype=torch.int32, device=DEVICE)
        for _ in range(scale):
            r = _rand(k, gen)
            u = 2 * u + (r >= a + b).to(torch.int32)
            v = 2 * v + (((r >= a) & (r < a + b)) | (r >= a + b + c)).to(torch.int32)
        e = torch.stack([perm[u.long()], perm[v.long()]], 1)
        flip = _rand(k, gen) < 0.5
        out[s:s + k] = torch.where(flip[:, None], e.flip(1), e)
    return out


def _chung_lu(sizes, pairs, gen):
    """Power-law graphs back to back: graph g has sizes[g] vertices (ids local to it) and pairs[g] draws
    whose endpoints follow weights (i + 1)^(-1 / (GAMMA - 1)), ids permuted inside each graph."""
    n = torch.as_tensor(sizes, device=DEVICE)
    E = torch.as_tensor(pairs, device=DEVICE)
    base = torch.cumsum(n, 0) - n
    total = int(n.sum())
    graph = torch.repeat_interleave(torch.arange(n.numel(), device=DEVICE), n)
    order = torch.argsort(graph.to(torch.float64) + _rand(total, gen, torch.float64))
    local = (order - base[graph]).to(torch.int32)
    p = 1.0 - 1.0 / (GAMMA - 1.0)
    out = torch.empty((int(E.sum()), 2), dtype=torch.int32, device=DEVICE)
    g = torch.repeat_interleave(torch.arange(n.numel(), device=DEVICE), E)
    for s in range(0, out.shape[0], 1 << 26):
        ge = g[s:s + (1 << 26)]
        top = (n[ge] + 1).to(torch.float64) ** p - 1.0
        for side in range(2):
            i = ((_rand(ge.numel(), gen, torch.float64) * top + 1.0) ** (1.0 / p)).long() - 1
            i = torch.minimum(i.clamp_(min=0), n[ge] - 1)
            out[s:s + (1 << 26), side] = local[base[ge] + i]
    return out


def _rgg(n, degree, gen):
    """Random geometric graph on the unit square, average degree about `degree`, each pair once."""
    r = math.sqrt(degree / (math.pi * n))
    side = max(1, int(1.0 / r))
    pos = _rand((n, 2), gen, torch.float64)
    ij = (pos * side).long().clamp_(max=side - 1)
    cell, order = torch.sort(ij[:, 0] * side + ij[:, 1])
    ij = ij[order]
    x, y = pos[order, 0], pos[order, 1]
    start = torch.searchsorted(cell, torch.arange(side * side + 1, device=DEVICE))
    me = torch.arange(n, device=DEVICE)
    parts = []
    for di, dj in ((0, 0), (0, 1), (1, -1), (1, 0), (1, 1)):   # own cell, then half of the eight around it
        ci, cj = ij[:, 0] + di, ij[:, 1] + dj
        inside = (ci < side) & (cj >= 0) & (cj < side)
        c = torch.where(inside, ci * side + cj, torch.zeros_like(ci))
        first = start[c] if (di, dj) != (0, 0) else me + 1
        count = torch.where(inside, start[c + 1] - first, torch.zeros_like(ci))
        u = torch.repeat_interleave(me, count)
        v = torch.arange(u.numel(), device=DEVICE) + (first - (torch.cumsum(count, 0) - count))[u]
        dx, dy = x[u] - x[v], y[u] - y[v]
        near = dx * dx + dy * dy <= r * r
        parts.append(torch.stack([order[u[near]], order[v[near]]], 1).to(torch.int32))
        del u, v, near, dx, dy
    return _shuffled(torch.cat(parts), gen)


def _vertices(case):
    return 1 << case["scale"] if case["graph"] == "rmat" else case["n"]


def _graph_sizes(case):
    """(vertices, pairs) of each graph of a queue or batch: pairs spread evenly over their logarithm."""
    G = case["graphs"]
    q = (np.arange(G) + 0.5) / G
    pairs = np.rint(case["lo"] * (case["hi"] / case["lo"]) ** q).astype(np.int64)
    return np.maximum(pairs // 8, 2), pairs


def _edges(case, gen):
    if case["graph"] == "rgg":
        return _rgg(case["n"], case["degree"], gen)
    n, pairs = _vertices(case), case["pairs"]
    if case["graph"] == "er" or case.get("distinct"):
        return _distinct(case, n, pairs, gen)
    return _draws(case, n, pairs, gen)


def _draws(case, n, pairs, gen):
    if case["graph"] == "rmat":
        return _rmat(case["scale"], pairs, gen)
    if case["graph"] == "chung_lu":
        return _chung_lu([n], [pairs], gen)
    return torch.randint(0, n, (pairs, 2), generator=gen, device=DEVICE, dtype=torch.int32)


def _distinct(case, n, pairs, gen):
    """`pairs` distinct vertex pairs of the family, without loops."""
    key = torch.empty(0, dtype=torch.int64, device=DEVICE)
    while key.numel() < pairs:
        e = _draws(case, n, pairs + pairs // 8 + 64, gen).long()
        lo, hi = torch.minimum(e[:, 0], e[:, 1]), torch.maximum(e[:, 0], e[:, 1])
        key = torch.unique(torch.cat([key, (lo * n + hi)[lo != hi]]))
    key = key[torch.randperm(key.numel(), generator=gen, device=DEVICE)[:pairs]]
    return _shuffled(torch.stack([key // n, key % n], 1), gen)


def _selector_samples(case, gen):
    """Bucket features as a counting call reports them, a strategy per bucket, the time at stake."""
    B = case["batch"]
    din = torch.randint(0, 15, (B,), generator=gen, device=DEVICE).float()
    dout = torch.randint(0, 16, (B,), generator=gen, device=DEVICE).float()
    logv = 20.0 * _rand(B, gen)                       # log2 of the bucket's vertices
    x = torch.stack([din / 14, dout / 15, (logv + 1) / 32, (logv + din) / 32, (logv + dout) / 32,
                     (logv + din + dout) / 48], 1).contiguous()
    label = torch.where(din >= 6, 2, torch.where(dout >= 4, 1, 0)).to(torch.int32)
    noise = torch.randint(0, 3, (B,), generator=gen, device=DEVICE, dtype=torch.int32)
    label = torch.where(_rand(B, gen) < 0.1, noise, label)
    weight = torch.sqrt(_rand(B, gen) * 4 + 0.01)
    return x, label.contiguous(), weight


def prepare(case, seed):
    gen = _generator(seed)
    state = {"case": case}
    if case["call"] == "selector" or case.get("select") == "learned":
        tc.selector_load(WEIGHTS, DEVICE)
    if case["call"] == "selector":
        state["samples"] = _selector_samples(case, gen)
        return state
    state["select"] = SELECT[case.get("select", "heuristic")]
    if case["call"] in ("queue", "batch"):
        nv, pairs = _graph_sizes(case)
        order = np.random.Generator(np.random.PCG64(seed)).permutation(nv.size)   # sizes arrive in any order
        nv, pairs = nv[order], pairs[order]
        state["edges"] = _chung_lu(nv, pairs, gen)
        state["offsets"] = np.concatenate([[0], np.cumsum(pairs)])
        state["vertices"] = nv.astype(np.int32)
        if case["call"] == "queue":
            off = state["offsets"]
            state["graphs"] = [(state["edges"][off[g]:off[g + 1]], int(nv[g])) for g in range(nv.size)]
            need = max(tc.workspace_size(e.shape[0], n, state["select"]) for e, n in state["graphs"])
            state["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEVICE)
            state["results"] = torch.zeros((nv.size, 2), dtype=torch.int64, device=DEVICE)
        return state
    state["edges"] = _edges(case, gen)
    state["n"] = _vertices(case)
    if case["call"] == "noalloc":
        state["result"] = torch.zeros(2, dtype=torch.int64, device=DEVICE)
        state["per_vertex"] = (torch.zeros(state["n"], dtype=torch.int64, device=DEVICE) if case["per_vertex"]
                               else None)
    return state


# ---------------------------------------------------------------- one pass
def run(state):
    case = state["case"]
    call = case["call"]
    if call == "selector":
        x, label, weight = state["samples"]
        logits = tc.selector_forward(x)
        grad, loss = tc.selector_gradient(x, label, weight)
        return logits, grad, loss
    if call == "batch":
        return tc.count_triangles_batch(state["edges"], state["offsets"], state["vertices"], select=state["select"])
    if call == "queue":
        for g, (edges, n) in enumerate(state["graphs"]):
            tc.count_triangles_async(edges, n, result=state["results"][g], select=state["select"],
                                     workspace=state["workspace"])
        return state["results"]
    edges, n, select = state["edges"], state["n"], state["select"]
    if call == "noalloc":
        tc.count_triangles_noalloc(edges, n, state["result"], per_vertex=state["per_vertex"], select=select)
        return (state["result"], state["per_vertex"]) if case["per_vertex"] else state["result"]
    if call == "clustering":
        return tc.clustering(edges, n, per_vertex=True, select=select)
    if call == "support":
        return tc.edge_support(edges, n, select=select)
    if call == "edge_counts":
        return tc.edge_counts(edges, n, select=select)
    if call == "csr":
        return tc.build_csr(edges, n)
    return tc.count_triangles(edges, n, per_vertex=case["per_vertex"], select=select)


# ---------------------------------------------------------------- work, reference
def work(case):
    """The pair list read once and the outputs written once; the selector's also its multiply-adds."""
    if case["call"] == "selector":
        B, params, macs = case["batch"], 1379, 6 * 32 + 32 * 32 + 32 * 3
        return {"bytes": 4 * (B * (6 + 1 + 1 + 3) + 2 * params), "flops": 2 * macs * B * 4}   # forward twice, backward
    if case["call"] in ("queue", "batch"):
        nv, pairs = _graph_sizes(case)
        return {"bytes": 8 * int(pairs.sum()) + 16 * case["graphs"], "flops": 0}
    n = _vertices(case)
    pairs = int(n * case["degree"] / 2) if case["graph"] == "rgg" else case["pairs"]
    out = {"count": 8 * n if case.get("per_vertex") else 0, "noalloc": 8 * n if case.get("per_vertex") else 0,
           "clustering": 16 * n, "support": 12 * pairs, "edge_counts": 12 * pairs, "csr": 12 * n + 4 * pairs}
    return {"bytes": 8 * pairs + out[case["call"]], "flops": 0}


def _triangles_per_vertex(edges, n):
    """t[v] and the simple-graph degrees: for every kept edge, each later neighbour of its lower end looked up."""
    e = edges.long()
    lo, hi = torch.minimum(e[:, 0], e[:, 1]), torch.maximum(e[:, 0], e[:, 1])
    key = torch.unique((lo * n + hi)[lo != hi])
    a, b = key // n, key % n
    deg = torch.bincount(a, minlength=n) + torch.bincount(b, minlength=n)
    place = torch.empty(n, dtype=torch.int64, device=DEVICE)
    place[torch.argsort(deg, stable=True)] = torch.arange(n, device=DEVICE)
    pa, pb = place[a], place[b]
    key, _ = torch.sort(torch.minimum(pa, pb) * n + torch.maximum(pa, pb))
    src, dst = key // n, key % n
    end = torch.cumsum(torch.bincount(src, minlength=n), 0)[src]
    later = end - 1 - torch.arange(key.numel(), device=DEVICE)
    t = torch.zeros(n, dtype=torch.int64, device=DEVICE)
    cuts = torch.cumsum(later, 0)
    first = 0
    while first < key.numel():
        done = int(cuts[first - 1]) if first else 0
        last = max(first + 1, int(torch.searchsorted(cuts, done + (1 << 25))))
        k = later[first:last]
        edge = torch.repeat_interleave(torch.arange(first, min(last, key.numel()), device=DEVICE), k)
        step = torch.arange(edge.numel(), device=DEVICE) - (torch.cumsum(k, 0) - k)[edge - first]
        w = dst[edge + 1 + step]
        want = dst[edge] * n + w
        at = torch.searchsorted(key, want).clamp_(max=key.numel() - 1)
        hit = key[at] == want
        for ends in (src[edge[hit]], dst[edge[hit]], w[hit]):
            t += torch.bincount(ends, minlength=n)
        first = last
    return t[place], deg


def exact(case, seed):
    if case["call"] == "selector":
        x, label, weight = (s.double() if s.is_floating_point() else s.long()
                            for s in _selector_samples(case, _generator(seed)))
        with open(WEIGHTS) as f:
            p = torch.tensor(json.load(f)["params"], dtype=torch.float32, device=DEVICE)
        cuts = [192, 32, 1024, 32, 96, 3]
        shapes = [(32, 6), (32,), (32, 32), (32,), (3, 32), (3,)]
        theta = []
        for part, shape in zip(torch.split(p, cuts), shapes):   # weights are used rounded to bfloat16, biases not
            part = part.to(torch.bfloat16) if len(shape) == 2 else part
            theta.append(part.double().reshape(shape).requires_grad_())
        w1, b1, w2, b2, w3, b3 = theta
        z = torch.relu(torch.relu(x @ w1.T + b1) @ w2.T + b2) @ w3.T + b3
        loss = (weight * torch.nn.functional.cross_entropy(z, label, reduction="none")).mean()
        grads = torch.autograd.grad(loss, theta)
        return z.detach(), torch.cat([g.reshape(-1) for g in grads]), float(loss.detach())
    if case["call"] == "clustering":
        n = _vertices(case)
        t, deg = _triangles_per_vertex(_edges(case, _generator(seed)), n)
        wedge = deg * (deg - 1) // 2
        coeff = torch.where(wedge > 0, t.double() / wedge.clamp(min=1).double(), torch.zeros(1, device=DEVICE).double())
        T, W = int(t.sum()) // 3, int(wedge.sum())
        return coeff, T, W, (3.0 * T / W if W else 0.0), t
    return None   # counts are whole numbers
