"""Performance cases of the graph beam-search library, through its public entry points.

A case is one piece of work that a program using the library does over and
over, or once at its start:

  search   a batch of queries on an index resident in HBM, through
           Index.search (device tensors or numpy arrays) or, for serving loops
           that must not allocate, gorio_search_noalloc;
  paged    a batch of queries on an index of which HBM holds only a page
           cache, nodes placed and queries admitted cluster by cluster;
  cluster  cluster_order: the placement computed before a paged index is built;
  build    an index built from host arrays and its first batch answered (what
           a program does when it starts, or takes a new index in).

Inputs: vectors of a Gaussian mixture (uint8 rows, or float32 rows of unit
length), queries of the same mixture, and a graph whose nodes have edges to the
nearest of a sample of their cluster and to random nodes.  Everything is drawn
on the GPU from the seed.  Sizes are those of the repository's own workloads
(10k and 1M nodes x 128 uint8, 96 float32; R = 32 and 64; L = 32, 64, 128) and
generic ones around them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2607_04415_amd as g

DEV = "cuda"
NO_EDGE = 0xFFFFFFFF
SAMPLE = 1024          # cluster members a node's near edges are chosen from
BLOCK = 256            # nodes (neighbours in cluster order) that share a sample
MODES = {"split": 0, "blocking": 1, "host": 2, "queue": 3}


# --------------------------------------------------------------------------- #
# the cases
# --------------------------------------------------------------------------- #
def _search(dtype, n, D, R, nq, L, W, k=10, via="search", layout="vectors", placed=False):
    return {"kind": "search", "dtype": dtype, "n": n, "D": D, "R": R, "nq": nq, "L": L, "W": W, "k": k,
            "via": via, "layout": layout, "placed": placed}


def _paged(dtype, n, D, R, nq, L, W, mode, cache, latency_us, clusters, oversub=1, k=10):
    return {"kind": "paged", "dtype": dtype, "n": n, "D": D, "R": R, "nq": nq, "L": L, "W": W, "k": k,
            "mode": mode, "cache": cache, "latency_us": latency_us, "clusters": clusters, "oversub": oversub}


def _cluster(dtype, n, D, clusters, iterations):
    return {"kind": "cluster", "dtype": dtype, "n": n, "D": D, "clusters": clusters, "iterations": iterations}


def _build(dtype, n, D, R, nq, L, W, layout="vectors", k=10):
    return {"kind": "build", "dtype": dtype, "n": n, "D": D, "R": R, "nq": nq, "L": L, "W": W, "k": k,
            "layout": layout, "placed": False}


def listed():
    return [
        # one user's query as it comes in: the smallest call, all latency
        dict(_search("u8", 1_000_000, 128, 64, 1, 64, 4), name="u8-one-query"),
        # a serving loop's small batch, into buffers it keeps
        dict(_search("f32", 200_000, 96, 64, 32, 64, 4, via="noalloc"), name="f32-serving-32"),
        # the small workload: 10k nodes, 1,000 queries
        dict(_search("u8", 10_000, 128, 32, 1000, 32, 4), name="u8-10k"),
        # the main workload: 1M nodes, 10,000 queries
        dict(_search("u8", 1_000_000, 128, 64, 10_000, 64, 4), name="u8-1m"),
        # the same index asked for higher recall, in a larger batch: the largest search
        dict(_search("u8", 1_000_000, 128, 64, 20_000, 128, 8), name="u8-1m-wide"),
        # the float32 workload's rows, frontier and beam (on a tenth of its nodes)
        dict(_search("f32", 1_000_000, 96, 64, 10_000, 128, 8), name="f32-1m"),
        # float32 rows of another length
        dict(_search("f32", 300_000, 128, 32, 5000, 64, 4), name="f32-d128"),
        # ragged rows in contiguous records placed by cluster, queries and answers in host memory
        dict(_search("u8", 300_000, 100, 48, 5000, 64, 4, via="host", layout="contiguous", placed=True),
             name="u8-d100-host"),
        # a tenth of the index in HBM, the GPU scheduler (parks a query on a missing page)
        dict(_paged("u8", 200_000, 128, 64, 1000, 64, 4, "split", 0.10, 0.0, 128), name="u8-paged-split"),
        # a tenth of a float32 index in HBM, 20 us per page, the GPU resume queue
        dict(_paged("f32", 100_000, 96, 64, 500, 64, 8, "queue", 0.10, 20.0, 64), name="f32-paged-queue"),
        # the placement of the main workload's index
        dict(_cluster("u8", 1_000_000, 128, 512, 4), name="u8-cluster-order"),
        # start of a program: a float32 index and its first batch
        dict(_build("f32", 1_000_000, 96, 32, 1000, 64, 4), name="f32-build"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search"] * 7 + ["paged", "paged", "cluster", "build"])
    dtype = rng.choice(["u8", "f32"])
    if dtype == "u8":
        D = rng.choice([128, 128, 4 * rng.randint(4, 64)])
    else:
        D = rng.choice([96, rng.randint(16, 256), 4 * rng.randint(4, 64)])
    R = rng.choice([32, 64, rng.randint(12, 96)])
    L = rng.choice([32, 64, 128, rng.randint(12, 200)])
    W = rng.choice([4, 8, rng.randint(1, 12)])
    k = min(L, rng.choice([10, 10, rng.randint(1, 100)]))
    vec = D * (1 if dtype == "u8" else 4)
    if kind == "search":
        # at most about the listed largest search's bytes, and a 512 MB index
        n = min(_log(rng, 5_000, 1_000_000), (512 << 20) // (vec + 4 * R))
        most = int(20_000 * 128 * 64 * 128 / ((L + W) * R * vec))
        nq = max(1, min(_log(rng, 1, 20_000), most))
        return _search(dtype, n, D, R, nq, L, W, k, via=rng.choice(["search", "search", "noalloc", "host"]),
                       layout=rng.choice(["vectors", "vectors", "contiguous"]), placed=rng.random() < 0.25)
    if kind == "paged":
        n = _log(rng, 20_000, 150_000)
        nq = max(16, int(100 * 64 / L))
        return _paged(dtype, n, D, R, nq, L, W, rng.choice(["split", "split", "blocking", "host", "queue"]),
                      rng.choice([0.05, 0.10, 0.20]), rng.choice([0.0, 20.0]), rng.randint(16, 128),
                      oversub=rng.choice([1, 4]), k=k)
    if kind == "cluster":
        return _cluster(dtype, min(_log(rng, 20_000, 1_000_000), (128 << 20) // vec), D, _log(rng, 16, 512),
                        rng.randint(1, 4))
    n = min(_log(rng, 20_000, 1_000_000), (512 << 20) // (vec + 4 * R))
    return _build(dtype, n, D, R, max(1, int(1000 * 64 / L)), L, W, layout=rng.choice(["vectors", "contiguous"]), k=k)


# --------------------------------------------------------------------------- #
# inputs
# --------------------------------------------------------------------------- #
def _mixture(gen, centres, count, dtype):
    """`count` rows of the mixture and the clusters they were drawn from."""
    C, D = centres.shape
    labels = torch.randint(C, (count,), generator=gen, device=DEV)
    out = torch.empty((count, D), dtype=torch.uint8 if dtype == "u8" else torch.float32, device=DEV)
    sigma = 20.0 if dtype == "u8" else 0.05
    for s in range(0, count, 1 << 18):
        c = labels[s:s + (1 << 18)]
        v = centres[c] + sigma * torch.randn((len(c), D), generator=gen, device=DEV)
        out[s:s + (1 << 18)] = v.round_().clamp_(0, 255).to(torch.uint8) if dtype == "u8" else v / v.norm(dim=1, keepdim=True)
    return labels, out


def _vectors(case, seed):
    """Vectors, their clusters, the generator and the mixture's centres."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    n, D, u8 = case["n"], case["D"], case["dtype"] == "u8"
    C = max(4, n // 4000)
    if u8:
        centres = 40.0 + 175.0 * torch.rand((C, D), generator=gen, device=DEV)
    else:
        centres = torch.randn((C, D), generator=gen, device=DEV)
        centres /= centres.norm(dim=1, keepdim=True)
    labels, x = _mixture(gen, centres, n, case["dtype"])
    return gen, centres, labels, x


def _graph(gen, x, labels, C, R):
    """n x R edges: half to the nearest of a sample of the node's cluster, half to random nodes.

    Distances are compared as whole numbers (float32 rows are scaled and
    rounded first) with the sample's position as the tie break, so that the
    same seed gives the same graph on every run."""
    n, D = x.shape
    near = R // 2
    order = torch.argsort(labels, stable=True)
    start = torch.searchsorted(labels[order].contiguous(), torch.arange(C + 1, device=DEV))
    xs = x[order].float() if x.dtype == torch.uint8 else (x[order] * 512.0).round_()
    if x.dtype == torch.uint8:
        xs -= 128.0   # keeps every sum below 2^24, where float32 adds whole numbers exactly
    norms = (xs * xs).sum(1)
    blocks = -(-n // BLOCK)
    graph = torch.randint(n, (n, R), generator=gen, device=DEV, dtype=torch.int32)
    lab = labels[order]
    # a sample for each block: members of the cluster of the block's middle node
    mid = lab[(torch.arange(blocks, device=DEV) * BLOCK + BLOCK // 2).clamp_(max=n - 1)]
    lo, size = start[mid], (start[mid + 1] - start[mid])
    pick = lo[:, None] + (torch.rand((blocks, SAMPLE), generator=gen, device=DEV) * size[:, None]).long().clamp_(max=n - 1)
    pick.clamp_(max=n - 1)
    col = torch.arange(SAMPLE, device=DEV, dtype=torch.int32)
    order32 = order.to(torch.int32)
    step = 512
    for b in range(0, blocks, step):
        p = pick[b:b + step]
        rows = torch.arange(b * BLOCK, (b + len(p)) * BLOCK, device=DEV).clamp_(max=n - 1).view(-1, BLOCK)
        dots = torch.bmm(xs[rows], xs[p].transpose(1, 2).contiguous())
        d = norms[rows][:, :, None] + norms[p][:, None, :] - 2.0 * dots
        d.masked_fill_(rows[:, :, None] == p[:, None, :], float(1 << 21))   # not the node itself
        key = d.clamp_(0, float((1 << 21) - 1)).to(torch.int32) * SAMPLE + col
        best = torch.topk(key, near, dim=2, largest=False, sorted=True).values % SAMPLE
        ids = order32[torch.gather(p, 1, best.view(len(p), -1).long())].view(-1, near)
        m = min(n - b * BLOCK, len(ids))
        graph[order[b * BLOCK:b * BLOCK + m], :near] = ids[:m]
    return graph


def _data(case, seed):
    gen, centres, labels, x = _vectors(case, seed)
    graph = _graph(gen, x, labels, len(centres), case["R"])
    _, q = _mixture(gen, centres, case["nq"], case["dtype"])
    return labels, x, graph, q


def _host(t):
    a = t.cpu().numpy()
    return a.view(np.uint32) if a.dtype == np.int32 else a


def prepare(case, seed):
    kind = case["kind"]
    if kind == "cluster":
        return {"case": case, "x": _host(_vectors(case, seed)[3])}
    labels, x, graph, q = _data(case, seed)
    xh, gh = _host(x), _host(graph)
    s = {"case": case, "q": q}
    if kind == "build":
        s.update(x=xh, graph=gh)
        return s
    if kind == "paged":
        n2s, centroids = g.cluster_order(xh, case["clusters"], 1)
        ix = g.Index(xh, gh, node_to_slot=n2s)
        info = ix.info
        ix.set_cache(max(int(case["cache"] * info["index_bytes"]), 256 * info["page_bytes"]))
        ix.set_query_order(centroids)
        ix.set_backing(latency_us=case["latency_us"], oversub=case["oversub"], mode=MODES[case["mode"]])
        ix.set_scheduler(query_waves=40)
        s["ix"] = ix
        return s
    n2s = None
    if case["placed"]:   # nodes cluster by cluster
        n2s = np.empty(case["n"], np.uint32)
        n2s[_host(torch.argsort(labels, stable=True))] = np.arange(case["n"], dtype=np.uint32)
    s["ix"] = g.Index(xh, gh, node_to_slot=n2s, vectors_first=case["layout"] == "vectors")
    if case["via"] == "host":
        s["q"] = _host(q)
    elif case["via"] == "noalloc":
        s["ids"] = torch.empty((case["nq"], case["k"]), dtype=torch.int32, device=DEV)
        s["dists"] = torch.empty((case["nq"], case["k"]), device=DEV,
                                 dtype=torch.int32 if case["dtype"] == "u8" else torch.float32)
    return s


# --------------------------------------------------------------------------- #
# one pass
# --------------------------------------------------------------------------- #
def run(s):
    c = s["case"]
    if c["kind"] == "cluster":
        n2s, centroids = g.cluster_order(s["x"], c["clusters"], c["iterations"])
        return {"node_to_slot": n2s, "centroids": centroids}
    if c["kind"] == "build":
        ix = g.Index(s["x"], s["graph"], vectors_first=c["layout"] == "vectors")
        ids, dists, _ = ix.search(s["q"], c["k"], c["L"], c["W"], stats=False)
        entry = ix.info["entry"]
        ix.close()
        return {"entry": entry, "ids": ids, "dists": dists}
    if c["kind"] == "search" and c["via"] == "noalloc":
        status = g.lib().gorio_search_noalloc(
            s["ix"]._h, s["q"].data_ptr(), c["nq"], c["k"], c["L"], c["W"], s["ids"].data_ptr(),
            s["dists"].data_ptr(), None, torch.cuda.current_stream().cuda_stream)
        if status != g.OK:
            raise RuntimeError(g.lib().gorio_last_error().decode())
        return {"ids": s["ids"], "dists": s["dists"]}
    ids, dists, _ = s["ix"].search(s["q"], c["k"], c["L"], c["W"], stats=False)
    return {"ids": ids, "dists": dists}


def work(case):
    """Bytes and operations of one pass: the queries, the answers, and per
    query the adjacency lists of its expanded nodes and the vectors of the
    nodes first met there (about L + W expansions, nearly all of whose edges
    lead to new nodes while these are few against the index)."""
    eb = 1 if case["dtype"] == "u8" else 4
    vec = case["D"] * eb
    n = case["n"]
    if case["kind"] == "cluster":
        steps = case["iterations"] + 1
        return {"bytes": n * vec + n * 4 + case["clusters"] * case["D"] * 4,
                "flops": 2.0 * n * case["clusters"] * case["D"] * steps + float(n * case["D"] * case["iterations"])}
    exp = min(n, case["L"] + case["W"])
    met = exp * case["R"]
    evals = n * (1.0 - math.exp(-met / n)) * 0.9
    per_query = exp * (4 + 4 * case["R"]) + evals * vec + vec + 8 * case["k"]
    out = {"bytes": case["nq"] * per_query, "flops": case["nq"] * evals * case["D"] * 3.0}
    if case["kind"] == "build":   # the vectors and edges in, the pages out
        out["bytes"] += 2.0 * n * (vec + 4 * case["R"])
        out["flops"] += 4.0 * n * case["D"]
    return out


def tolerance(case):
    """Answers are whole numbers (ids, uint8 distances, slots), and the library's
    float32 distances and centroids are sums in a stated order with every step
    rounded, equal to a plain sequential loop's: all of it is exact."""
    return "exact"


# --------------------------------------------------------------------------- #
# the same in 64 bits
# --------------------------------------------------------------------------- #
def _medoid64(x):
    n = len(x)
    if x.dtype == torch.uint8:
        c = torch.div(x.sum(0, dtype=torch.int64) + n // 2, n, rounding_mode="floor").double()
    else:
        c = (x.sum(0, dtype=torch.float64) / n).float().double()
    best, at = math.inf, 0
    for s in range(0, n, 1 << 17):
        d = (x[s:s + (1 << 17)].double() - c).square().sum(1)
        m = d.min()
        if float(m) < best:
            best, at = float(m), s + int((d == m).nonzero()[0])
    return at


def _search64(x, graph, q, entry, k, L, W):
    """The search's stated loop, a batch of queries at a time, distances in float64."""
    n, R = graph.shape
    nq = len(q)
    graph = graph.long()
    xd = x.double()
    ids_out = torch.full((nq, k), -1, dtype=torch.int64, device=DEV)
    d_out = torch.full((nq, k), math.inf, dtype=torch.float64, device=DEV)
    step = max(1, min(nq, int(4e9 / max(n, W * R * x.shape[1] * 8))))
    for s in range(0, nq, step):
        qd = q[s:s + step].double()
        m = len(qd)
        seen = torch.zeros((m, n), dtype=torch.bool, device=DEV)
        seen[:, entry] = True
        fd = torch.full((m, L), math.inf, dtype=torch.float64, device=DEV)
        fi = torch.full((m, L), n, dtype=torch.int64, device=DEV)
        fx = torch.zeros((m, L), dtype=torch.bool, device=DEV)
        fd[:, 0] = (qd - xd[entry]).square().sum(1)
        fi[:, 0] = entry
        live = torch.arange(m, device=DEV)
        while len(live):
            a, b, e = fd[live], fi[live], fx[live]
            todo = ~e & (b < n)
            sel = todo & (todo.cumsum(1) <= W)
            go = sel.any(1)
            live, a, b, e, sel = live[go], a[go], b[go], e[go], sel[go]
            if not len(live):
                break
            e = e | sel
            at = torch.argsort((~sel).to(torch.int8), dim=1, stable=True)[:, :W]
            took = torch.gather(sel, 1, at)
            nb = graph[torch.gather(b, 1, at).clamp(max=n - 1)]
            ok = (took[:, :, None] & (nb >= 0)).reshape(len(live), -1)
            nb = nb.reshape(len(live), -1).masked_fill(~ok, n).sort(1).values
            first = torch.ones_like(ok)
            first[:, 1:] = nb[:, 1:] != nb[:, :-1]
            safe = nb.clamp(max=n - 1)
            new = first & (nb < n) & ~seen[live[:, None], safe]
            rows, cols = new.nonzero(as_tuple=True)
            v = nb[rows, cols]
            seen[live[rows], v] = True
            nd = torch.full(nb.shape, math.inf, dtype=torch.float64, device=DEV)
            nd[rows, cols] = (xd[v] - qd[live[rows]]).square().sum(1)
            a = torch.cat([a, nd], 1)
            b = torch.cat([b, torch.where(new, nb, n)], 1)
            e = torch.cat([e, torch.zeros_like(new)], 1)
            by = torch.argsort(b, dim=1, stable=True)
            by = torch.gather(by, 1, torch.argsort(torch.gather(a, 1, by), dim=1, stable=True))[:, :L]
            fd[live], fi[live], fx[live] = torch.gather(a, 1, by), torch.gather(b, 1, by), torch.gather(e, 1, by)
        ids_out[s:s + step] = torch.where(fi[:, :k] < n, fi[:, :k], -1)
        d_out[s:s + step] = fd[:, :k]
    return ids_out, d_out


def exact(case, seed):
    if case["kind"] == "cluster":
        x = _vectors(case, seed)[3].double()
        n, K = len(x), case["clusters"]
        c = x[torch.arange(K, device=DEV) * n // K]
        key = None
        for it in range(case["iterations"] + 1):
            key = torch.cat([((c * c).sum(1) - 2.0 * (x[s:s + 65536] @ c.T)).argmin(1) for s in range(0, n, 65536)])
            if it == case["iterations"]:
                break
            cnt = torch.bincount(key, minlength=K)
            sums = torch.zeros_like(c).index_add_(0, key, x)
            c = torch.where(cnt[:, None] > 0, sums / cnt.clamp(min=1)[:, None], c)
        n2s = torch.empty(n, dtype=torch.int64, device=DEV)
        n2s[torch.argsort(key, stable=True)] = torch.arange(n, device=DEV)
        return {"node_to_slot": n2s, "centroids": c}
    if case["nq"] * (case["L"] + case["W"]) * case["R"] * case["D"] > 1.2e10:   # over about 20 seconds
        return None
    _, x, graph, q = _data(case, seed)
    entry = _medoid64(x)
    ids, dists = _search64(x, graph, q, entry, case["k"], case["L"], case["W"])
    if case["dtype"] == "u8":
        dists = torch.where(torch.isinf(dists), 2147483647.0, dists).long()
    out = {"ids": ids, "dists": dists}
    if case["kind"] == "build":
        out["entry"] = entry
    return out
