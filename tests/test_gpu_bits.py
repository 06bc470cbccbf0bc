"""The bit-mask fixpoints (hop levels on any graph, every algebra on unit
weights) at their edges: 1, 2 and 4 groups side by side and padded ones, rows
cut into slices, more levels than eight planes hold, isolated vertices, graphs
of fewer vertices than a bitmap word, directed graphs, weights that are all 1,
and a second call on the same graph."""
import numpy as np
import pytest

import oracle
from paper_1609_07008_amd import graphgen as gg
from tests.test_gpu_fixpoint import host, mfbc, oracle_rows, same_values, unweighted  # noqa: F401

pytestmark = pytest.mark.gpu


def ones():
    g = gg.er_graph(700, 9, 3)
    return gg.Graph(g.n, g.row_ptr, g.col, np.ones(g.arcs, np.int32), "ones")


FORMS = {
    "rmat11_unw": lambda: gg.rmat_graph(11, 16, 5),
    "star3000": lambda: gg.star_graph(3000),
    "path700": lambda: gg.path_graph(700),
    "pair": lambda: gg.path_graph(2),
    "ones": ones,
    "rmat12_w255": lambda: gg.rmat_graph(12, 16, 7, wrange=(1, 255)),
    "directed": lambda: gg.directed_rmat_graph(10, 8, 12, wrange=(1, 50)),
    "unpacked": lambda: gg.er_graph(300, 12, 7, (1, 6_000_000)),
}


@pytest.mark.parametrize("nb", [1, 64, 65, 130, 200, 256, 300, 500])
@pytest.mark.parametrize("name", list(FORMS))
def test_hop_levels(mfbc, name, nb):  # noqa: F811
    g = FORMS[name]()
    src = np.random.default_rng(nb).integers(0, g.n, size=nb).astype(np.int32)
    print(f"[bits] {name} nb={nb}", flush=True)
    unw = type(g)(g.n, g.row_ptr, g.col, None)
    ref = oracle.brandes(unw, src)["dist"]
    dg = mfbc.DeviceGraph(g, directed=name == "directed")
    for _ in range(2):
        h, products = dg.fixpoint(src, "bfs")
        assert np.array_equal(host(h, mfbc.INF_DIST), ref)
        assert products == int(ref.max()) + 1
    dg.set_plan(run_arcs=64, run_verts=5, heavy=30, slice=7)
    h, products = dg.fixpoint(src, "bfs")
    assert np.array_equal(host(h, mfbc.INF_DIST), ref) and products == int(ref.max()) + 1
    dg.close()


@pytest.mark.parametrize("op", ["sssp", "widest", "resist"])
@pytest.mark.parametrize("name", ["rmat11_unw", "path700", "pair", "ones", "star3000"])
def test_algebras_on_unit_weights(mfbc, name, op):  # noqa: F811
    g = FORMS[name]()
    src = np.random.default_rng(3).integers(0, g.n, size=70).astype(np.int32)
    dg = mfbc.DeviceGraph(g)
    d, products = dg.fixpoint(src, op)
    if op == "sssp":
        ref = oracle.brandes(g, src)["dist"]
        assert np.array_equal(host(d, mfbc.INF_DIST), ref) and products == int(ref.max()) + 1
    else:
        want, n = oracle_rows(g, src, op)
        assert same_values(d, want, op) and products == n
    dg.close()
