"""Calls whose frontier outlives the products that fit 16 bits, on graphs whose
rows are long enough to start in them: they go on in 32 bits from the state
reached (k_quad_widen).  One to four groups a row of words, padded groups,
split rows, path counts and frontier multiplicities that are escaped in
both forms, in one and in none; columns that are done before, and components
that the landmarks do not reach.  Distances and product counts bit-exact, path
counts within 1e-12, dependencies within 1e-10; against the CPU oracle, the
traced call (in 32 bits throughout) for the product counts."""
import numpy as np
import pytest

import oracle
from paper_1609_07008_amd import graphgen as gg
from tests.test_gpu_fixpoint import host
from tests.test_gpu_parity import DELTA_TOL, SIGMA_TOL, mfbc, rel_close, torch  # noqa: F401
from tests.test_gpu_quad import beside, weighted

pytestmark = pytest.mark.gpu


def cliques(count, size, lo, hi, seed):
    """`count` cliques in a row, each joined to the next by two edges."""
    rng = np.random.default_rng(seed)
    a, b = np.triu_indices(size, 1)
    base = np.arange(count)[:, None] * size
    u, v = [(base + a).ravel()], [(base + b).ravel()]
    for k in range(2):
        u.append(base[:-1, 0] + k)
        v.append(base[1:, 0] + size - 1 - k)
    u, v = np.concatenate(u), np.concatenate(v)
    return gg.csr_from_edges(count * size, u, v, rng.integers(lo, hi + 1, u.size), f"cliques{count}x{size}")


def directed(g, seed):
    """Both arcs of every edge, of different weights."""
    u, v, w = g.edges()
    rng = np.random.default_rng(seed)
    tail, head = np.concatenate([u, v]), np.concatenate([v, u])
    order = np.lexsort((head, tail))
    rp = np.zeros(g.n + 1, np.int64)
    rp[1:] = np.cumsum(np.bincount(tail, minlength=g.n))
    return gg.DiGraph(g.n, rp, head[order].astype(np.int32),
                      rng.integers(1, w.max() + 1, tail.size).astype(np.int32), g.name)


FORMS = {
    "cliques": lambda: cliques(70, 62, 1, 255, 1),                     # long paths, few ties
    "cliques_even": lambda: cliques(70, 62, 255, 255, 2),              # every weight alike: ties everywhere
    "cliques_w399": lambda: cliques(70, 62, 1, 399, 3),                # 40 products with counts, 160 without
    "cliques_w1638": lambda: cliques(70, 62, 1, 1638, 4),              # none with counts, 40 without
    "diamonds": lambda: beside(weighted(gg.diamond_chain(60), 255, 255, 1)),    # counts double every other product
    "layers": lambda: beside(weighted(gg.layered_bipartite(90, 5), 255, 255, 1)),   # 5^89 paths
    "directed": lambda: directed(cliques(70, 62, 1, 255, 5), 6),
}


@pytest.mark.parametrize("name", list(FORMS))
def test_products_past_16_bits(torch, mfbc, name):  # noqa: F811
    g = FORMS[name]()
    assert g.arcs >= 1 << 18
    dg = mfbc.DeviceGraph(g, directed=name == "directed")
    rng = np.random.default_rng(5)
    src = rng.integers(0, g.n, size=330).astype(np.int32)
    src[::3] = rng.integers(0, 150, size=src[::3].size)                # many at one end
    ref = oracle.brandes(g, src)
    out = torch.empty(g.n, dtype=torch.float64, device="cuda")
    for nb in (1, 64, 65, 128, 129, 200, 256, 300, 330):
        lam = oracle.brandes(g, src[:nb], per_source=False)["lambda"]
        for plan in ({}, dict(run_arcs=64, run_verts=5, heavy=30, slice=16)):
            print(f"[widen] {name} arcs={g.arcs} nb={nb} plan={plan}", flush=True)
            dg.set_plan(**plan)
            f = dg.forward(src[:nb])
            assert np.array_equal(host(f["dist"], mfbc.INF_DIST), ref["dist"][:nb])
            rel_close(f["sigma"].cpu().numpy(), ref["sigma"][:nb], SIGMA_TOL, "sigma")
            products = dg.forward(src[:nb], trace=True, frontiers=False)["products"]
            assert f["products"] == products > 40
            d, again = dg.fixpoint(src[:nb], "sssp")
            assert np.array_equal(host(d, mfbc.INF_DIST), ref["dist"][:nb]) and again <= products
            rel_close(dg.bc(src[:nb], nb).cpu().numpy(), lam, DELTA_TOL, "one batch")
            rel_close(dg.bc(src[:nb], 70).cpu().numpy(), lam, DELTA_TOL, "batches of 70")
    dg.set_lanes(3)
    rel_close(dg.bc(src, 64).cpu().numpy(), lam, DELTA_TOL, "three lanes")
    parts = [src[:3], src[3:80], src[80:]]
    for o, p in zip(dg.bc_requests(parts, 128), parts):
        rel_close(o.cpu().numpy(), oracle.brandes(g, p, per_source=False)["lambda"], DELTA_TOL, "request")
    dg.bc_noalloc(torch.from_numpy(src).cuda(), 64, out)
    rel_close(out.cpu().numpy(), lam, DELTA_TOL, "no allocation")
    for x, o in zip((src, src[:50]), mfbc.bc_many([dg, dg], [src, src[:50]])):
        rel_close(o.cpu().numpy(), oracle.brandes(g, x, per_source=False)["lambda"], DELTA_TOL, "batched")
    dg.close()
