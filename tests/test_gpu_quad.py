"""The 16-bit products behind mfbc_forward and the shortest-distance fixpoint
(graphs of 2^18 arcs and more) at their edges: one and two words a lane, padded
groups, saturated multiplicities (ties by the thousand, counts up to 2^60) in
runs and in slices, weights at the ends of the range that fits, frontiers that
outlive it, columns whose component the landmarks do not reach, directed arcs,
weights that are not packed.  Distances and product counts bit-exact, path
counts within 1e-12; the oracle on all of them, the traced call (in 32 bits) for
the product counts."""
import numpy as np
import pytest

import oracle
from paper_1609_07008_amd import graphgen as gg
from tests.test_gpu_fixpoint import host, mfbc, oracle_rows  # noqa: F401
from tests.test_gpu_parity import SIGMA_TOL, rel_close

pytestmark = pytest.mark.gpu


def weighted(g, lo, hi, seed):
    u, v, _ = g.edges()
    w = np.random.default_rng(seed).integers(lo, hi + 1, u.size)
    return gg.csr_from_edges(g.n, u, v, w, g.name)


def beside(g, seed=3):
    """g next to a component large enough for the 16-bit products."""
    wide = gg.rmat_graph(13, 26, seed, wrange=None if g.w is None else (1, g.max_weight))
    u, v, w = g.edges()
    a, b, x = wide.edges()
    return gg.csr_from_edges(g.n + wide.n, np.concatenate([u, a + g.n]), np.concatenate([v, b + g.n]),
                             None if g.w is None else np.concatenate([w, x]), g.name)


NB = [1, 64, 65, 128, 129, 200, 256, 300]
FORMS = {
    "rmat14_w255": (lambda: gg.rmat_graph(14, 16, 6, wrange=(1, 255)), NB),
    "rmat14_w3": (lambda: gg.rmat_graph(14, 16, 7, wrange=(1, 3)), [64, 200]),
    "rmat14_unw": (lambda: gg.rmat_graph(14, 16, 5), [64, 130, 256]),
    "er3000_w399": (lambda: gg.er_graph(3000, 100, 9, (1, 399)), [70, 200]),     # widest with counts
    "er3000_w1638": (lambda: gg.er_graph(3000, 100, 9, (1, 1638)), [70, 200]),   # widest without
    "er3000_w1639": (lambda: gg.er_graph(3000, 100, 9, (1, 1639)), [70]),
    "bipartite": (lambda: gg.complete_bipartite_graph(300, 500), [65, 256]),
    "layers": (lambda: gg.layered_bipartite(6, 170), [65, 200]),                 # 170^5 paths
    "layers_w": (lambda: weighted(gg.layered_bipartite(5, 190), 2, 2, 1), [130]),
    "diamonds": (lambda: beside(gg.diamond_chain(60)), NB),                      # 2^60 paths
    "diamonds_w9": (lambda: beside(weighted(gg.diamond_chain(30), 9, 9, 1)), [130]),
    "path90_w255": (lambda: beside(gg.path_graph(90, w=255)), [65, 130]),        # outlives 56 products
    "path300_w255": (lambda: beside(gg.path_graph(300, w=255)), [65, 130]),      # and 256
    "star": (lambda: gg.star_graph(140_000), [3, 130]),
    "hubs": (lambda: gg.rmat_graph(13, 48, 9, (0.7, 0.1, 0.1, 0.1), (1, 100)), [130]),
    "directed": (lambda: gg.directed_rmat_graph(14, 24, 12, wrange=(1, 250)), [65, 200]),
    "unpacked": (lambda: gg.er_graph((1 << 21) + 5, 0.14, 7, (1, 399)), [3]),
}


@pytest.mark.parametrize("name", list(FORMS))
def test_distances_and_path_counts(mfbc, name):  # noqa: F811
    make, nbs = FORMS[name]
    g = make()
    dg = mfbc.DeviceGraph(g, directed=name == "directed")
    rng = np.random.default_rng(5)
    src = rng.integers(0, g.n, size=max(nbs)).astype(np.int32)
    if name.startswith(("diamonds", "path")):      # half the columns on the small part
        src[::2] = rng.integers(0, 60, size=src[::2].size)
    ref = oracle.brandes(g, src)
    for nb in nbs:
        print(f"[quad] {name} arcs={g.arcs} nb={nb}", flush=True)
        for plan in ({}, dict(run_arcs=64, run_verts=5, heavy=30, slice=16)):
            dg.set_plan(**plan)
            f = dg.forward(src[:nb])
            assert np.array_equal(host(f["dist"], mfbc.INF_DIST), ref["dist"][:nb])
            rel_close(f["sigma"].cpu().numpy(), ref["sigma"][:nb], SIGMA_TOL, "sigma")
            assert f["products"] == dg.forward(src[:nb], trace=True, frontiers=False)["products"]
            d, products = dg.fixpoint(src[:nb], "sssp")
            assert np.array_equal(host(d, mfbc.INF_DIST), ref["dist"][:nb])
    if g.n < 10_000:
        few = src[:6]
        assert dg.fixpoint(few, "sssp")[1] == oracle_rows(g, few, "sssp")[1]
    dg.close()


@pytest.mark.parametrize("size", ["small", "large"])
def test_bad_source_is_refused_and_the_next_call_is_right(mfbc, size):  # noqa: F811
    g = gg.rmat_graph(11, 16, 6, wrange=(1, 255)) if size == "small" else FORMS["rmat14_w255"][0]()
    dg = mfbc.DeviceGraph(g)
    src = np.arange(70, dtype=np.int32)
    bad = src.copy()
    bad[66] = g.n
    ref = oracle.brandes(g, src)
    f = dg.forward(src)
    for call in (lambda: dg.forward(bad), lambda: dg.fixpoint(bad, "sssp"), lambda: dg.fixpoint(bad, "bfs"),
                 lambda: dg.fixpoint(bad, "widest"), lambda: dg.bc(bad, 64), lambda: dg.bc(bad, 32),
                 lambda: dg.backward(bad, f["dist"], f["sigma"])):
        with pytest.raises(mfbc.MfbcError) as e:
            call()
        assert e.value.code == mfbc.MFBC_EINVAL and "outside" in str(e.value)
        assert np.array_equal(host(dg.forward(src)["dist"], mfbc.INF_DIST), ref["dist"])
    dg.close()
