"""Centrality with its forward products in 16 bits on the shortest-path core:
one group and odd numbers of groups, padded columns, saturated path counts,
rows cut into slices, frontiers that outlive the products that fit (the 32-bit
products then start over), weights that leave them no room at all, several
lanes, request lists.  Against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_1609_07008_amd import graphgen as gg
from tests.test_gpu_parity import DELTA_TOL, mfbc, rel_close, torch  # noqa: F401
from tests.test_gpu_quad import beside

pytestmark = pytest.mark.gpu


def weighted(g, w):
    u, v, _ = g.edges()
    return gg.csr_from_edges(g.n, u, v, np.full(u.size, w), g.name)


def bundles(a, b):
    """Two bundles of parallel two-arc paths in a row: a * b shortest paths end to end."""
    mid = np.arange(a), a + 1 + np.arange(b)
    ends = np.full(a, a + b + 1), np.full(a, a), np.full(b, a), np.full(b, a + b + 2)
    return gg.csr_from_edges(a + b + 3, np.concatenate([mid[0], mid[0], mid[1], mid[1]]), np.concatenate(ends), None,
                             f"bundles{a}x{b}")


FORMS = {
    "er1024": lambda: gg.er_graph(1024, 8, 3, (1, 100)),
    "rmat10_w255": lambda: gg.rmat_graph(10, 16, 6, wrange=(1, 255)),
    "rmat11_unw": lambda: gg.rmat_graph(11, 16, 5),                 # rows that every column has reached
    "hubs_unw": lambda: gg.rmat_graph(12, 48, 9, (0.7, 0.1, 0.1, 0.1)),
    "directed_unw": lambda: gg.directed_rmat_graph(10, 24, 12),
    "diamonds": lambda: gg.diamond_chain(60),                       # 2^60 paths
    "diamonds_w9": lambda: weighted(gg.diamond_chain(30), 9),
    "paths65534": lambda: bundles(217, 302),
    "paths65535": lambda: bundles(255, 257),
    "paths65536": lambda: bundles(256, 256),
    "layers": lambda: gg.layered_bipartite(6, 60),                  # 60^5 paths
    "path57_w255": lambda: gg.path_graph(57, w=255),                # the last that fits, in 56 products
    "path90_w255": lambda: gg.path_graph(90, w=255),                # outlives them
    "er300_w399": lambda: gg.er_graph(300, 20, 9, (1, 399)),        # 40 products fit
    "er300_w400": lambda: gg.er_graph(300, 20, 9, (1, 400)),        # too few do
    "hubs": lambda: gg.rmat_graph(12, 48, 9, (0.7, 0.1, 0.1, 0.1), (1, 100)),
    "directed": lambda: gg.directed_rmat_graph(10, 24, 12, wrange=(1, 250)),
    "unpacked": lambda: gg.er_graph(300, 40, 7, (1, 6_000_000)),
}


@pytest.mark.parametrize("name", list(FORMS))
def test_centrality_against_the_oracle(torch, mfbc, name):  # noqa: F811
    g = FORMS[name]()
    dg = mfbc.DeviceGraph(g, directed=name.startswith("directed"))
    src = np.random.default_rng(5).integers(0, g.n, size=330).astype(np.int32)
    if name.startswith("paths"):
        src[[0, 70, 129]] = g.n - 1, g.n - 2, g.n - 1               # the ends of the bundles
    out = torch.empty(g.n, dtype=torch.float64, device="cuda")
    for nb in (1, 64, 65, 128, 129, 330):
        print(f"[bc16] {name} arcs={g.arcs} nb={nb}", flush=True)
        want = oracle.brandes(g, src[:nb], per_source=False)["lambda"]
        for plan in ({}, dict(run_arcs=64, run_verts=5, heavy=30, slice=16)):
            dg.set_plan(**plan)
            rel_close(dg.bc(src[:nb], nb).cpu().numpy(), want, DELTA_TOL, "one batch")
            rel_close(dg.bc(src[:nb], 70).cpu().numpy(), want, DELTA_TOL, "batches of 70")
    for lanes in (1, 3):
        dg.set_lanes(lanes)
        rel_close(dg.bc(src, 64).cpu().numpy(), want, DELTA_TOL, f"{lanes} lanes")
    dg.set_lanes(0)
    dg.bc_noalloc(torch.from_numpy(src).cuda(), 128, out)
    rel_close(out.cpu().numpy(), want, DELTA_TOL, "no allocation")
    parts = [src[:3], src[3:80], src[80:]]
    for o, p in zip(dg.bc_requests(parts, 128), parts):
        rel_close(o.cpu().numpy(), oracle.brandes(g, p, per_source=False)["lambda"], DELTA_TOL, "request")
    dg.close()


@pytest.mark.parametrize("name", ["paths65534", "paths65535", "paths65536"])
def test_path_counts_where_they_stop_fitting(mfbc, name):  # noqa: F811
    g = beside(FORMS[name]())
    dg = mfbc.DeviceGraph(g)
    small = FORMS[name]().n
    for nb in (3, 130, 200):
        src = np.arange(small - nb, small, dtype=np.int32)
        print(f"[bc16] {name} forward nb={nb}", flush=True)
        ref = oracle.brandes(g, src)
        f = dg.forward(src)
        assert np.array_equal(f["sigma"].cpu().numpy(), ref["sigma"])
    dg.close()
