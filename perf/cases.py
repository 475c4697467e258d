"""Performance cases: what users of the library run, over the range they run it on.

Every case is one call through the public Python entry points on a synthetic
graph made on the GPU from the seed:

  exact       nk_bc_exact, every vertex as a source
  batch       a captured NkBatchPlan over many small graphs, run once
  sources     nk_bc_sources / _linear / _bisect over k sampled sources
  directed    nk_bc_directed with the in-arc CSR at hand
  weighted    nk_bc_weighted, integer weights on both arcs of every edge
  edge        nk_edge_bc: edge and vertex scores of one run
  closeness   nk_closeness_sampled over k sources
  pairs       nk_bc_pair_sample, the epsilon-delta estimate

Graph kinds: "er" (uniform random edges), "ba" (preferential attachment),
"rmat" (R-MAT 0.57/0.19/0.19/0.05, folded onto n vertices), "cl" (Chung-Lu,
exponent 2.5).  `deg` is the number of generated edges per vertex (self-loops
and repeats are dropped).
"""
import math

import numpy as np
import torch

import paper_1403_3005_amd as nk

DEV = "cuda"


def listed():
    return [
        # the smallest call: one network of a few hundred vertices (a social circle, a
        # regulatory network), exact scores; launches and latency are all of it
        {"name": "exact_er_300", "op": "exact", "kind": "er", "n": 300, "deg": 3},
        # the exact benchmark graph, G(2000, 10000)
        {"name": "exact_er_2000", "op": "exact", "kind": "er", "n": 2000, "deg": 5},
        # exact scores of a scale-free network of ordinary size (an internet map, a
        # collaboration network), an odd vertex count
        {"name": "exact_ba_9973", "op": "exact", "kind": "ba", "n": 9973, "deg": 4},
        # a study over many networks: a batch of graphs kept as a plan, run again
        {"name": "batch_16", "op": "batch", "kind": "mixed", "n": 1000, "n_hi": 25000, "deg": 4, "graphs": 16},
        # the headline benchmark: 4096 sampled sources on R-MAT scale 20
        {"name": "sources_rmat20_4096", "op": "sources", "kind": "rmat", "n": 1 << 20, "deg": 16, "k": 4096,
         "est": "plain"},
        # the interactive query of the serving workload: a quick estimate from 64 sources
        {"name": "sources_rmat18_64", "op": "sources", "kind": "rmat", "n": 1 << 18, "deg": 16, "k": 64,
         "est": "plain"},
        # a large sparse network without hubs, the upper end of the batched workload
        {"name": "sources_er200k_1024", "op": "sources", "kind": "er", "n": 200_000, "deg": 4, "k": 1024,
         "est": "plain"},
        # pair sampling with its guarantee on a power-law graph of a million vertices
        {"name": "pairs_cl_1m", "op": "pairs", "kind": "cl", "n": 1_000_000, "deg": 10, "eps": 0.01},
        # a directed web-like graph, transpose kept beside it
        {"name": "directed_rmat18_512", "op": "directed", "kind": "rmat", "n": 1 << 18, "deg": 16, "k": 512},
        # weighted shortest paths (travel costs), weights 1..64
        {"name": "weighted_rmat17_256", "op": "weighted", "kind": "rmat", "n": 1 << 17, "deg": 16, "k": 256},
        # edge scores for sparsification and community splits
        {"name": "edge_rmat17_512", "op": "edge", "kind": "rmat", "n": 1 << 17, "deg": 16, "k": 512},
        # sampled closeness of a large network
        {"name": "closeness_rmat18_1024", "op": "closeness", "kind": "rmat", "n": 1 << 18, "deg": 16, "k": 1024},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["exact", "exact", "batch", "sources", "sources", "sources", "directed", "weighted", "edge",
                     "closeness", "pairs"])
    if op == "exact":
        return {"op": op, "kind": rng.choice(["er", "ba", "rmat"]), "n": _log_uniform(rng, 200, 20000),
                "deg": rng.choice([2, 3, 4, 6])}
    if op == "batch":
        return {"op": op, "kind": "mixed", "n": _log_uniform(rng, 300, 2000), "n_hi": _log_uniform(rng, 4000, 25000),
                "deg": rng.choice([3, 4, 5]), "graphs": _log_uniform(rng, 4, 24)}
    if op == "pairs":
        return {"op": op, "kind": rng.choice(["cl", "rmat", "ba"]), "n": _log_uniform(rng, 10000, 1_000_000),
                "deg": rng.choice([4, 8, 10]), "eps": rng.choice([0.05, 0.02, 0.01])}
    kind = rng.choice(["er", "ba", "rmat"])
    n = _log_uniform(rng, 5000, 1 << 19)
    deg = rng.choice([4, 8, 16]) if kind == "rmat" else rng.choice([3, 4, 6])
    # arcs x sources at most an eighth of the largest listed case's (a weighted run a further eighth)
    most = (4096 * 16 * (1 << 20)) // (64 if op == "weighted" else 8)
    k = max(16, min(_log_uniform(rng, 16, 2048), n, most // (n * deg)))
    case = {"op": op, "kind": kind, "n": n, "deg": deg, "k": k}
    if op == "sources":
        case["est"] = rng.choice(["plain", "plain", "linear", "bisect"])
    return case


# ------------------------------------------------------------------ inputs --


def _arcs_er(n, deg, g):
    e = n * deg
    return torch.randint(0, n, (e,), generator=g, device=DEV), torch.randint(0, n, (e,), generator=g, device=DEV)


def _arcs_rmat(n, deg, g):
    scale = max(1, math.ceil(math.log2(n)))
    e = n * deg
    u = torch.zeros(e, dtype=torch.int64, device=DEV)
    v = torch.zeros(e, dtype=torch.int64, device=DEV)
    for _ in range(scale):
        r = torch.rand(e, generator=g, device=DEV)
        u = 2 * u + (r >= 0.76)                                          # (0.57 + 0.19)
        v = 2 * v + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95)).long()
    return u % n, v % n


def _arcs_ba(n, deg, g):
    # slot 2e is edge e's new vertex, slot 2e + 1 a copy of a uniform earlier slot
    e = (n - 1) * deg
    new = 1 + torch.arange(e, device=DEV) // deg
    first = 2 * deg * ((new - 1))                                        # slots filled before this vertex
    pick = (torch.rand(e, generator=g, device=DEV, dtype=torch.float64) * first).long()
    ptr = torch.arange(2 * e, device=DEV)
    ptr[1::2] = torch.where(first > 0, pick, torch.zeros_like(pick))
    ptr[1] = 0
    for _ in range(64):                                                  # pointer jumping to an even slot
        nxt = ptr[ptr]
        if bool((nxt == ptr).all()):
            break
        ptr = nxt
    val = 1 + (ptr // 2) // deg
    val[1:2 * deg:2] = 0                                                 # the first new vertex joins vertex 0
    return new, torch.where(ptr[1::2] % 2 == 0, val[1::2], torch.zeros_like(new))


def _arcs_cl(n, deg, g):
    w = (n / (torch.arange(n, device=DEV, dtype=torch.float64) + 1.0)) ** (2.0 / 3.0)
    c = torch.cumsum(w, 0)
    e = n * deg
    pick = [torch.searchsorted(c, torch.rand(e, generator=g, device=DEV, dtype=torch.float64) * c[-1]) for _ in "uv"]
    return pick[0].clamp_(max=n - 1), pick[1].clamp_(max=n - 1)


_ARCS = {"er": _arcs_er, "rmat": _arcs_rmat, "ba": _arcs_ba, "cl": _arcs_cl}


def _csr(n, u, v):
    keep = u != v
    key = torch.unique(u[keep] * n + v[keep])
    src, dst = key // n, key % n
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    return rowptr.int(), dst.int()


def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _graph(case, g):
    u, v = _ARCS[case["kind"]](case["n"], case["deg"], g)
    if case["op"] == "directed":
        return _csr(case["n"], u, v)
    if case["op"] == "edge":                                             # a fixed number of edges: scores come per arc
        n, keep = case["n"], u != v
        key = torch.unique(torch.minimum(u, v)[keep] * n + torch.maximum(u, v)[keep])
        key = key[torch.randperm(key.numel(), generator=g, device=DEV)[: _edges(case)]]
        u, v = key // n, key % n
    return _csr(case["n"], torch.cat([u, v]), torch.cat([v, u]))


def _edges(case):
    return int(case["n"] * case["deg"] * 0.6)


def _batch_sizes(case):
    lo, hi, count = case["n"], case["n_hi"], case["graphs"]
    return [int(round(math.exp(math.log(lo) + (math.log(hi) - math.log(lo)) * i / max(1, count - 1))))
            for i in range(count)]


def _tails(rowptr):
    n = rowptr.numel() - 1
    return torch.repeat_interleave(torch.arange(n, device=DEV), (rowptr[1:] - rowptr[:-1]).long())


def prepare(case, seed):
    g = _generator(seed)
    op = case["op"]
    if op == "batch":
        graphs = [_graph({"op": op, "kind": "ba" if i % 2 else "er", "n": n, "deg": case["deg"]}, g)
                  for i, n in enumerate(_batch_sizes(case))]
        vtx = np.cumsum([0] + [rp.numel() - 1 for rp, _ in graphs])
        arc = np.cumsum([0] + [ci.numel() for _, ci in graphs])
        plan = nk.NkBatchPlan(vtx, arc, torch.cat([rp for rp, _ in graphs]), torch.cat([ci for _, ci in graphs]))
        return {"op": op, "plan": plan, "graphs": graphs}
    rowptr, colidx = _graph(case, g)
    s = {"op": op, "rowptr": rowptr, "colidx": colidx, "n": case["n"], "seed": seed}
    if "k" in case:
        s["sources"] = torch.randperm(case["n"], generator=g, device=DEV)[: case["k"]].int()
        s["scale"] = case["n"] / case["k"]
    if op == "sources":
        s["est"] = case["est"]
    if op == "pairs":
        s["eps"] = case["eps"]
    if op == "directed":
        s["trowptr"], s["tcolidx"] = _csr(case["n"], colidx.long(), _tails(rowptr))
    if op == "weighted":
        u, v = _tails(rowptr), colidx.long()
        key = torch.minimum(u, v) * case["n"] + torch.maximum(u, v)
        salt = int(torch.randint(1, 1 << 30, (1,), generator=g, device=DEV))
        h = (key ^ salt) * 0x9E3779B97F4A7C1 & 0x7FFFFFFFFFFFFFFF
        s["weights"] = (1 + (h ^ (h >> 29)) % 64).int()
    return s


def run(s):
    op = s["op"]
    if op == "exact":
        return nk.nk_bc_exact(s["rowptr"], s["colidx"])
    if op == "batch":
        return s["plan"].run()
    if op == "pairs":
        bc, counts, r, vd = nk.nk_bc_pair_sample(s["rowptr"], s["colidx"], s["eps"], 0.1, s["seed"])
        return {"bc": bc, "counts": counts, "samples": r, "vd": vd}
    if op == "sources":
        if s["est"] == "plain":
            return nk.nk_bc_sources(s["rowptr"], s["colidx"], s["sources"], s["scale"])
        call = nk.nk_bc_sources_linear if s["est"] == "linear" else nk.nk_bc_sources_bisect
        return call(s["rowptr"], s["colidx"], s["sources"], 2 * s["scale"])
    if op == "directed":
        return nk.nk_bc_directed(s["rowptr"], s["colidx"], s["sources"], s["scale"], s["trowptr"], s["tcolidx"])
    if op == "weighted":
        return nk.nk_bc_weighted(s["rowptr"], s["colidx"], s["weights"], s["sources"], s["scale"])
    if op == "edge":
        ebc, bc = nk.nk_edge_bc(s["rowptr"], s["colidx"], s["sources"], s["scale"])
        return {"edge": ebc, "vertex": bc}
    return nk.nk_closeness_sampled(s["rowptr"], s["colidx"], s["sources"])


def work(case):
    """The graph read once and the scores written once; per source and edge, one addition
    of a path count and one of a dependency term (or one distance step for closeness)."""
    sizes = _batch_sizes(case) if case["op"] == "batch" else [case["n"]]
    arcs = [n * case["deg"] * (1 if case["op"] == "directed" else 2) for n in sizes]
    if case["op"] == "edge":
        arcs = [2 * _edges(case)]
    byts = sum(4 * (n + 1) + 4 * m + 8 * n for n, m in zip(sizes, arcs))
    if case["op"] == "weighted":
        byts += 4 * arcs[0]
    if case["op"] == "directed":
        byts += 4 * (case["n"] + 1) + 4 * arcs[0]
    if case["op"] == "edge":
        byts += 8 * arcs[0]
    if case["op"] == "pairs":
        # about six vertices on a path, and each sampled pair drawn and counted
        r = 0.5 / case["eps"] ** 2 * 6
        return {"bytes": byts + 4 * case["n"], "flops": 12 * r}
    per_source = sum(m * (case["k"] if "k" in case else n) for n, m in zip(sizes, arcs))
    return {"bytes": byts, "flops": per_source * (0.5 if case["op"] == "closeness" else 2)}


# -------------------------------------------------- the same in plain torch --


def _brandes(rowptr, colidx, sources, est="plain", weights=None, undirected_edges=False):
    """(sum over sources of dependencies, per-arc terms, distance sums), float64.

    Distances by relaxing all arcs until nothing changes, path counts and
    dependencies by as many sweeps over the shortest-path arcs as the
    longest of them has arcs, for a block of sources at a time.
    """
    n = rowptr.numel() - 1
    u, v = _tails(rowptr), colidx.long()
    m = v.numel()
    w = torch.ones(m, 1, device=DEV, dtype=torch.float64) if weights is None else weights.double()[:, None]
    bc = torch.zeros(n, device=DEV, dtype=torch.float64)
    ebc = torch.zeros(m, device=DEV, dtype=torch.float64) if undirected_edges else None
    far = torch.zeros(n, device=DEV, dtype=torch.float64)
    width = max(1, min(sources.numel(), (1 << 27) // max(m, n, 1)))
    for s in torch.split(sources.long(), width):
        b = s.numel()
        col = torch.arange(b, device=DEV)
        dist = torch.full((n, b), math.inf, device=DEV, dtype=torch.float64)
        dist[s, col] = 0.0
        vi = v[:, None].expand(m, b)
        while m:
            new = dist.scatter_reduce(0, vi, dist[u] + w, "amin")
            if torch.equal(new, dist):
                break
            dist = new
        far += torch.where(torch.isfinite(dist), dist, torch.zeros_like(dist)).sum(1)
        if est == "distances":
            continue
        dag = (torch.isfinite(dist[u]) & (dist[u] + w == dist[v])).double()
        root = torch.zeros(n, b, device=DEV, dtype=torch.float64)
        root[s, col] = 1.0
        sigma = root.clone()
        hops = 0
        while True:
            new = root.clone().index_add_(0, v, sigma[u] * dag)
            if torch.equal(new, sigma):
                break
            sigma = new
            hops += 1
        inv = torch.where(sigma > 0, 1.0 / sigma, torch.zeros_like(sigma))
        ratio = dag * sigma[u] * inv[v]

        def dependencies(target, factor=None):
            """delta with `target` (n x b) the weight of each vertex as a path end."""
            delta = torch.zeros_like(dist)
            for _ in range(hops):
                delta = torch.zeros_like(dist).index_add_(0, u, ratio * (target + delta)[v])
                if factor is not None:
                    delta = delta * factor
            return delta

        ones = torch.isfinite(dist).double()
        if est == "linear":
            d = torch.where(torch.isfinite(dist), dist, torch.zeros_like(dist))
            delta = dependencies(ones, d / (d + 1.0))
        elif est == "bisect":
            # the far half of every path: v counts for targets t with 2 d(v) > d(t), half at equality
            delta = torch.zeros_like(dist)
            deep = int(dist[torch.isfinite(dist)].max())
            for t in range(1, deep + 1):
                part = dependencies((dist == t).double())
                delta += part * ((2 * dist > t).double() + 0.5 * (2 * dist == t).double())
        else:
            delta = dependencies(ones)
        if ebc is not None:
            term = (ratio * (ones + delta)[v]).sum(1)
            ebc += term
        delta[s, col] = 0.0
        bc += delta.sum(1)
    if ebc is not None:
        order = torch.argsort(v * n + u)                                  # arc (u, v) next to its reverse
        ebc = ebc + ebc[order]
    return bc, ebc, far


def exact(case, seed):
    if case["op"] == "pairs":
        return None
    if case["op"] == "batch":
        if sum(n * n * case["deg"] for n in _batch_sizes(case)) > 2e9:
            return None
        s = prepare(case, seed)
        return torch.cat([_brandes(rp, ci, torch.arange(rp.numel() - 1, device=DEV))[0] for rp, ci in s["graphs"]])
    k = case.get("k", case["n"])
    if case["kind"] in ("rmat", "cl") and case["n"] * case["deg"] * k > 1e8:
        return None                                                      # adds into the hubs' rows take too long
    if case["n"] * case["deg"] * k * (8 if case.get("est") == "bisect" else 3 if case["op"] == "weighted" else 1) > 1.3e9:
        return None
    s = prepare(case, seed)
    src = s.get("sources", torch.arange(case["n"], device=DEV))
    scale = s.get("scale", 1.0)
    if case["op"] == "closeness":
        f = _brandes(s["rowptr"], s["colidx"], src, "distances")[2] * (case["n"] / k)
        return torch.where(f > 0, (case["n"] - 1) / f, torch.zeros_like(f))
    bc, ebc, _ = _brandes(s["rowptr"], s["colidx"], src, case.get("est", "plain"), s.get("weights"),
                          case["op"] == "edge")
    if case.get("est") in ("linear", "bisect"):
        return bc * 2 * scale
    if case["op"] == "edge":
        return {"edge": ebc * scale, "vertex": bc * scale}
    return bc * scale
