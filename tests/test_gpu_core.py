"""The shortest-path core (arcs that no landmark shows to be too long) at the
sizes and forms where its construction can go wrong: both orientations of a
directed graph, rows cut into slices, components no landmark reaches, arcs
exactly as long as the walk around them, weights too wide for packed arcs, the
caller's order, and paths longer than the landmark run.  Every entry point
that runs on it against the CPU oracle."""
import numpy as np
import pytest

import oracle
from oracle.frontier import backward_products
from paper_1609_07008_amd import graphgen as gg
from tests.test_gpu_parity import DELTA_TOL, mfbc, rel_close, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def ties():
    """Every arc (i, i + 2) weighs what the two steps around it weigh, or one more."""
    n = 600
    i = np.arange(n - 1)
    j = np.arange(n - 2)
    rng = np.random.default_rng(4)
    step = rng.integers(1, 40, n - 1)
    far = rng.integers(2, n - 3, 4000)
    a = np.concatenate([i, j, 0 * far])
    b = np.concatenate([i + 1, j + 2, far])
    w = np.concatenate([step, step[:-1] + step[1:] + rng.integers(0, 2, n - 2), rng.integers(1, 4000, 4000)])
    key, at = np.unique(a * n + b, return_index=True)
    return gg.csr_from_edges(n, key // n, key % n, w[at], "ties")


def two_parts():
    g = gg.rmat_graph(9, 16, 21, wrange=(1, 200))
    u, v, w = g.edges()
    return gg.csr_from_edges(2 * g.n + 3, np.concatenate([u, u + g.n]), np.concatenate([v, v + g.n]),
                             np.concatenate([w, w[::-1]]), "two_parts")


def long_path():
    """A path far longer than the landmark run, with heavy short cuts."""
    n = 900
    i = np.arange(n - 1)
    rng = np.random.default_rng(8)
    j = np.unique(rng.integers(0, n - 40, 2600))
    d = rng.integers(2, 40, j.size)
    return gg.csr_from_edges(n, np.concatenate([i, j]), np.concatenate([i + 1, j + d]),
                             np.concatenate([np.full(n - 1, 3), rng.integers(1, 120, j.size)]), "long_path")


FORMS = {
    "rmat11_w255": lambda: gg.rmat_graph(11, 16, 6, wrange=(1, 255)),
    "er500_k120": lambda: gg.er_graph(500, 120, 3, (1, 255)),
    "er60_k40": lambda: gg.er_graph(60, 40, 5, (1, 1000)),           # fewer vertices than landmarks
    "hubs": lambda: gg.rmat_graph(13, 32, 9, (0.7, 0.1, 0.1, 0.1), (1, 100)),   # rows of several slices
    "unpacked": lambda: gg.er_graph(300, 40, 7, (1, 6_000_000)),     # column and weight exceed 32 bits
    "ties": ties,
    "two_parts": two_parts,
    "long_path": long_path,
    "directed": lambda: gg.directed_rmat_graph(11, 16, 12, wrange=(1, 250)),
}


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("name", list(FORMS))
def test_core_gives_the_oracle_results(torch, mfbc, name, keep):  # noqa: F811
    from paper_1609_07008_amd.serve import ColumnServer
    g = FORMS[name]()
    print(f"[core] {name} n={g.n} arcs={g.arcs} keep_order={keep}", flush=True)
    dg = mfbc.DeviceGraph(g, keep_order=keep)
    src = np.random.default_rng(11).choice(g.n, min(g.n, 150), replace=False).astype(np.int32)
    ref = oracle.brandes(g, src)
    for batch in (64, 150):
        rel_close(dg.bc(src, batch).cpu().numpy(), ref["lambda"], DELTA_TOL, f"lambda batch {batch}")
    f = dg.forward(src)
    b = dg.backward(src, f["dist"], f["sigma"], trace=True)
    rel_close(b["delta"].cpu().numpy(), ref["delta"], DELTA_TOL, "delta")
    assert np.array_equal(b["step"].cpu().numpy(), ref["height"])
    assert b["products"] == backward_products(ref["height"], src)
    parts = [src[:7], src[7:]]
    want = [oracle.brandes(g, p, per_source=False)["lambda"] for p in parts]
    for o, w in zip(dg.bc_requests(parts, 128), want):
        rel_close(o.cpu().numpy(), w, DELTA_TOL, "request")
    for width in (64, 128):
        o = mfbc.bc_many([dg], [src], job_width=width)[0]
        rel_close(o.cpu().numpy(), ref["lambda"], DELTA_TOL, f"batched {width}")
    server = ColumnServer(dg, 192)
    cols = server.admit(src)
    while server.active_columns():
        server.step_launch()
        server.step_finish()
    out = torch.zeros(g.n, dtype=torch.float64, device="cuda")
    server.harvest_bc(np.sort(cols), [out] * src.size)
    rel_close(out.cpu().numpy(), ref["lambda"], DELTA_TOL, "served")
    server.close()
    dg.set_plan(run_arcs=64, run_verts=3, heavy=40, slice=16)       # many slices, in both views
    rel_close(dg.bc(src, 150).cpu().numpy(), ref["lambda"], DELTA_TOL, "lambda, other plan")
    dg.close()
