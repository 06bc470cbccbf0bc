"""The calls that stand for this framework's use, with inputs made on the GPU.

Every case is one call (or, for the served form, one request loop) through the
public entry points on a graph that is already resident, the way a program
uses them: the graph is loaded once, sources arrive as a device array, results
stay on the device.  The families and their parameters are those of the
benchmark and the tests: R-MAT graphs (edge factor 16, weights 1..255 or
none), uniform random graphs, directed R-MAT graphs, and mixed suites of small
graphs.

A case holds
  kind       bc, forward, backward, fixpoint, requests, noalloc, many, serve
  family     rmat (undirected), drmat (directed), er (uniform), mixed (many)
  n, k       vertices and average degree (rmat, drmat: k = 2 x / 1 x edge factor)
  wmax       weights uniform in 1..wmax, 0 = unweighted
  nsrc       source columns (0 = every vertex), batch (columns per batch)
  op         fixpoint algebra; count = graphs of a mixed suite
"""
import math

import numpy as np
import torch

from paper_1609_07008_amd import autotune, graphgen, mfbc
from paper_1609_07008_amd.serve import ColumnServer

OPS = ("sssp", "bfs", "widest", "resist")


def _case(name, kind, family, n, k, wmax, nsrc, batch, op="", count=1):
    c = dict(kind=kind, family=family, n=n, k=k, wmax=wmax, nsrc=nsrc, batch=batch, op=op, count=count)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: distances and path counts of one column group on a graph of
        # a few hundred vertices, where launches and round trips are all there is
        _case("forward_er300_s64", "forward", "er", 300, 6, 20, 64, 64),
        # exact centrality of a small network, every vertex a source, small batches
        _case("bc_er1024_all_b64", "bc", "er", 1024, 8, 100, 0, 64),
        # approximate centrality of an unweighted social-network-like graph, wide batches
        _case("bc_rmat16_unw_s2048_b512", "bc", "rmat", 1 << 16, 32, 0, 2048, 512),
        # the headline: one batch on the weighted scale-20 power-law graph, the largest
        _case("bc_rmat20_w255_s256_b256", "bc", "rmat", 1 << 20, 32, 255, 256, 256),
        # a dense uniform graph: few products, very many ties
        _case("bc_er32k_k512_w255_s256_b256", "bc", "er", 32768, 512, 255, 256, 256),
        # a directed graph of odd size with ragged batches
        _case("bc_drmat100k_w100_s300_b150", "bc", "drmat", 100_003, 16, 100, 300, 150),
        # distances and path counts of a ragged batch, handed out source by source
        _case("forward_rmat18_w255_s200", "forward", "rmat", 1 << 18, 32, 255, 200, 200),
        # dependencies from given distances and path counts
        _case("backward_rmat18_w255_s130", "backward", "rmat", 1 << 18, 32, 255, 130, 130),
        # shortest distances and hop levels alone (the generic monoid product)
        _case("sssp_rmat19_w255_s256", "fixpoint", "rmat", 1 << 19, 32, 255, 256, 256, "sssp"),
        _case("bfs_rmat19_s256", "fixpoint", "rmat", 1 << 19, 32, 255, 256, 256, "bfs"),
        # the batched form: exact centrality of many small graphs of uneven sizes in one launch
        _case("many32_mixed", "many", "mixed", 6000, 48, 100, 0, 64, count=32),
        # the served form: requests of uneven sizes in the columns of one server
        _case("serve_rmat16_w255_c256", "serve", "rmat", 1 << 16, 32, 255, 230, 256),
    ]


# Most (arc, column) pairs of one pass: those of the largest listed case.
_MOST = (1 << 25) * 256


def draw(rng):
    """One more case: sizes log-uniform over the listed range, any kind, weight range and batch."""
    def logu(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("bc", "bc", "bc", "forward", "backward", "fixpoint", "fixpoint", "requests",
                       "noalloc", "many", "serve"))
    if kind == "many":
        return _case("", "many", "mixed", logu(400, 6000), rng.randint(6, 48), 100, 0, 64,
                     count=rng.randint(5, 32))
    family = rng.choice(("rmat", "rmat", "er", "er", "drmat"))
    n = logu(257, 900) if kind == "noalloc" else logu(300, 1 << 19)
    k = logu(4, 48)
    if family == "er" and kind != "noalloc" and n < 40_000:
        k = logu(3, 256)
    k = min(k, n // 4)
    wmax = rng.choice((0, 10, 100, 255, 255, 4000))
    nsrc = logu(1, 520) if kind in ("bc", "requests") else logu(1, 256)
    nsrc = max(1, min(nsrc, n // 2, _MOST // (2 * n * k)))
    batch = rng.choice((64, 100, 128, 150, 256, 512)) if kind == "bc" else 256 if kind == "requests" else \
        64 if kind == "noalloc" else max(64, nsrc) if kind != "serve" else -(-nsrc // 64) * 64
    return _case("", kind, family, n, k, wmax, nsrc, batch, rng.choice(OPS) if kind == "fixpoint" else "")


# ------------------------------------------------------------------------------ inputs
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _pairs(family, n, k, gen):
    """Head and tail of more arcs than wanted, loops and repeats among them."""
    half = max(1, n * k // (1 if family == "drmat" else 2))
    if family == "er":
        half = int(half * 1.05) + 16
        return (torch.randint(0, n, (half,), generator=gen, device="cuda"),
                torch.randint(0, n, (half,), generator=gen, device="cuda"))
    scale = max(1, math.ceil(math.log2(n)))
    u = torch.zeros(half, dtype=torch.int64, device="cuda")
    v = torch.zeros(half, dtype=torch.int64, device="cuda")
    for _ in range(scale):      # quadrants (0.57, 0.19, 0.19, 0.05), as in graphgen
        r = torch.rand(half, generator=gen, device="cuda")
        u = 2 * u + (r >= 0.76)
        v = 2 * v + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    keep = (u < n) & (v < n)
    perm = torch.randperm(n, generator=gen, device="cuda")
    return perm[u[keep]], perm[v[keep]]


def _graph(family, n, k, wmax, gen):
    """The graph in host memory (CSR, columns ascending), as mfbc_load_graph takes it."""
    u, v = _pairs(family, n, k, gen)
    if family != "drmat":
        u, v = torch.minimum(u, v), torch.maximum(u, v)
    key = torch.unique((u * n + v)[u != v])
    u, v = key // n, key % n
    w = torch.randint(1, wmax + 1, (key.numel(),), generator=gen, device="cuda") if wmax else None
    if family != "drmat":
        order = torch.argsort(torch.cat((key, v * n + u)))
        u, v = torch.cat((u, v))[order], torch.cat((v, u))[order]
        w = torch.cat((w, w))[order] if wmax else None
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(u, minlength=n), 0)
    host = (rp.cpu().numpy(), v.to(torch.int32).cpu().numpy(),
            w.to(torch.int32).cpu().numpy() if wmax else None)
    return (graphgen.DiGraph if family == "drmat" else graphgen.Graph)(n, *host)


def _sources(g, nsrc, gen):
    """Vertices with out-arcs, without repeats; every vertex if nsrc is 0."""
    if not nsrc:
        return torch.arange(g.n, dtype=torch.int32, device="cuda")
    cand = torch.from_numpy(np.flatnonzero(np.diff(g.row_ptr) > 0)).cuda()
    pick = torch.randperm(cand.numel(), generator=gen, device="cuda")[:nsrc]
    return cand[pick].to(torch.int32).contiguous()


def _suite(case, gen):
    """Graphs of a mixed suite: n spread log-uniformly up to case["n"], degrees up to case["k"],
    both families; the sizes are the case's, the graphs the seed's."""
    out = []
    for i in range(case["count"]):
        n = int(round(200 * (case["n"] / 200) ** ((0.31 + i * 0.6180339887) % 1.0)))
        k = 4 + int((0.77 + i * 0.7548776662) % 1.0 * (case["k"] - 4))
        out.append(_graph("rmat" if i % 2 else "er", n, k, case["wmax"], gen))
    return out


def _requests(case):
    """Lengths of the source lists of a request mix: uneven, odd ones among them."""
    left, out, part = case["nsrc"], [], 7
    while left > 0:
        out.append(min(left, part))
        left -= out[-1]
        part = part * 2 + 3
    return out


def _inputs(case, seed):
    gen = _generator(seed)
    if case["kind"] == "many":
        gs = _suite(case, gen)
        return gs, [_sources(g, 0, gen) for g in gs]
    g = _graph(case["family"], case["n"], case["k"], case["wmax"], gen)
    return [g], [_sources(g, case["nsrc"], gen)]


def prepare(case, seed):
    gs, srcs = _inputs(case, seed)
    s = dict(case=case, graphs=[mfbc.DeviceGraph(g) for g in gs], srcs=srcs)
    dg, src, kind = s["graphs"][0], srcs[0], case["kind"]
    if kind == "backward":
        s["fwd"] = dg.forward(src)
    elif kind == "many":
        cache = autotune.load_cache()
        autotune.apply_many_plans(s["graphs"], cache)
        s["cfg"] = autotune.many_config(cache)
    elif kind in ("requests", "serve"):
        cuts = np.cumsum(_requests(case))[:-1]
        s["lists"] = [x for x in np.split(src.cpu().numpy(), cuts) if x.size]
        if kind == "serve":
            s["server"] = ColumnServer(dg, case["batch"])
    elif kind == "noalloc":
        s["out"] = torch.empty(dg.n, dtype=torch.float64, device="cuda")
    return s


def run(state):
    case, dg, src = state["case"], state["graphs"][0], state["srcs"][0]
    kind = case["kind"]
    if kind == "bc":
        return dg.bc(src, case["batch"])
    if kind == "forward":
        return dg.forward(src)
    if kind == "backward":
        return dg.backward(src, state["fwd"]["dist"], state["fwd"]["sigma"])
    if kind == "fixpoint":
        return dg.fixpoint(src, case["op"])
    if kind == "requests":
        return dg.bc_requests(state["lists"], case["batch"])
    if kind == "noalloc":
        return dg.bc_noalloc(src, case["batch"], state["out"])
    if kind == "many":
        return mfbc.bc_many(state["graphs"], state["srcs"], **state["cfg"])[:64]
    # served: admit every list, step until its columns are done, add them into its sum
    server = state["server"]
    outs = [torch.zeros(dg.n, dtype=torch.float64, device="cuda") for _ in state["lists"]]
    dest = {}
    for x, out in zip(state["lists"], outs):
        for c in server.admit(x):
            dest[int(c)] = out
    cols = sorted(dest)
    while server.active_columns():
        server.step_launch()
        server.step_finish()
    server.harvest_bc(np.array(cols, dtype=np.int32), [dest[c] for c in cols])
    return outs


def work(case):
    """The adjacency, the sources and what is handed in read once, the results written
    once; for every (arc, column) an addition and a comparison, and for centrality the
    same again for the sums along the way back."""
    k, n = case["k"], case["n"]
    if case["kind"] == "many":      # n log-uniform in [200, n]: the means of n and n * n
        span = math.log(n / 200)
        m1, m2 = (n - 200) / span, (n * n - 200 * 200) / (2 * span)
        kk, cnt = (k + 4) / 2, case["count"]
        return {"bytes": cnt * m1 * (kk * 8 + 20), "flops": cnt * 4.0 * m2 * kk}
    cols = case["nsrc"] or n
    arcs = float(n * k)
    b = arcs * (8 if case["wmax"] and case["op"] != "bfs" else 4) + 8.0 * n + 4.0 * cols
    b += {"forward": 12.0, "backward": 20.0, "fixpoint": 4.0}.get(case["kind"], 0.0) * n * cols
    if case["kind"] in ("requests", "serve"):
        b += 8.0 * n * len(_requests(case))
    elif case["kind"] in ("bc", "noalloc"):
        b += 8.0 * n
    return {"bytes": b, "flops": arcs * cols * (2.0 if case["kind"] in ("fixpoint", "forward") else 4.0)}


# ------------------------------------------------------------------------------ 64 bits
_FAR = 1 << 40


def _relax(u, v, w, src, n, unit=False):
    """Shortest distances int64[n][columns] by relaxing every arc until nothing changes."""
    d = torch.full((n, src.numel()), _FAR, dtype=torch.int64, device="cuda")
    d[src.long(), torch.arange(src.numel(), device="cuda")] = 0
    step = torch.ones_like(w) if unit else w
    while True:
        new = d.index_reduce(0, v, d[u] + step[:, None], "amin")
        new = torch.where(new >= _FAR, _FAR, new)
        if torch.equal(new, d):
            return d
        d = new


def _best(u, v, w, src, n, op):
    """Bottleneck widths (0: none) or least sums of 1/w (inf: none), as _relax."""
    cols = torch.arange(src.numel(), device="cuda")
    if op == "widest":
        d = torch.zeros((n, src.numel()), dtype=torch.int64, device="cuda")
        d[src.long(), cols] = mfbc.INF_DIST
        f, how = (lambda x: torch.minimum(x, w[:, None])), "amax"
    else:
        d = torch.full((n, src.numel()), math.inf, dtype=torch.float64, device="cuda")
        d[src.long(), cols] = 0.0
        f, how = (lambda x: x + (1.0 / w.double())[:, None]), "amin"
    while True:
        new = d.index_reduce(0, v, f(d[u]), how)
        if torch.equal(new, d):
            return d
        d = new


def _paths(u, v, w, d, src):
    """Path counts float64[n][columns] and the tight arcs, from the distances."""
    cols = torch.arange(src.numel(), device="cuda")
    tight = ((d[u] + w[:, None] == d[v]) & (d[u] < _FAR)).double()
    seed = torch.zeros(d.shape, dtype=torch.float64, device="cuda")
    seed[src.long(), cols] = 1.0
    s, depth = seed, 0
    while True:
        new = seed.index_add(0, v, tight * s[u])
        depth += 1
        if torch.equal(new, s):
            return s, tight, depth
        s = new


def _dependencies(u, v, s, tight, depth, src):
    inv = torch.where(s > 0, 1.0 / s, 0.0)
    z = torch.zeros_like(s)
    for _ in range(depth):
        z = torch.zeros_like(s).index_add(0, u, tight * (z + inv)[v])
    delta = z * s
    delta[src.long(), torch.arange(src.numel(), device="cuda")] = 0.0
    return delta


def _brandes(g, src, chunk, want):
    n = g.n
    rows = torch.from_numpy(np.diff(g.row_ptr)).cuda()
    u = torch.repeat_interleave(torch.arange(n, device="cuda"), rows)
    v = torch.from_numpy(g.col.astype(np.int64)).cuda()
    w = torch.ones_like(v) if g.w is None else torch.from_numpy(g.w.astype(np.int64)).cuda()
    for i in range(0, src.numel(), chunk):
        x = src[i:i + chunk]
        if want in ("widest", "resist"):
            yield _best(u, v, w, x, n, want)
            continue
        d = _relax(u, v, w, x, n, want == "bfs")
        if want in ("sssp", "bfs"):
            yield d
            continue
        s, tight, depth = _paths(u, v, w, d, x)
        yield (d, s) if want == "forward" else _dependencies(u, v, s, tight, depth, x)


def exact(case, seed):
    """The same results from their definitions: relaxation to a fixpoint in int64, path
    counts and dependencies as float64 sums over the shortest-path arcs."""
    cols = case["nsrc"] or case["n"]
    if case["kind"] == "many":
        if work(case)["flops"] > 6e9:
            return None
    elif float(case["n"]) * case["k"] * cols > 1.2e9:
        return None
    gs, srcs = _inputs(case, seed)
    chunk = max(1, int(1.5e8 / max(g.col.size for g in gs)))

    def rows(parts):
        return torch.cat([p.t() for p in parts]).contiguous()

    def total(g, src):
        out = torch.zeros(g.n, dtype=torch.float64, device="cuda")
        for p in _brandes(g, src, chunk, "delta"):
            out += p.sum(1)
        return out

    g, src, kind = gs[0], srcs[0], case["kind"]
    if kind in ("bc", "noalloc"):
        return total(g, src)
    if kind == "many":
        return [total(a, b) for a, b in zip(gs, srcs)][:64]
    if kind in ("requests", "serve"):
        cuts = tuple(int(x) for x in np.cumsum(_requests(case))[:-1])
        return [total(g, x) for x in torch.tensor_split(src, cuts) if x.numel()]
    if kind == "backward":
        return {"delta": rows(_brandes(g, src, chunk, "delta")), "products": None}
    if kind == "forward":
        parts = list(_brandes(g, src, chunk, "forward"))
        d = rows(p[0] for p in parts)
        return {"dist": torch.where(d >= _FAR, mfbc.INF_DIST, d).to(torch.int32),
                "sigma": rows(p[1] for p in parts), "products": None}
    got = rows(_brandes(g, src, chunk, case["op"]))
    if case["op"] == "resist":
        return got, None
    return torch.where(got >= _FAR, mfbc.INF_DIST, got).to(torch.int32), None
