"""The batched form's two ways of running (few graphs one after another on
streams, many small ones in one persistent launch) on the same graphs: ragged
sizes, a handle listed twice, an empty source list, a decomposition set by the
caller, each arc encoding.  Against the CPU oracle; statistics of the handles
stay those of their own last call."""
import numpy as np
import pytest

import oracle
from paper_1609_07008_amd import graphgen as gg
from tests.test_gpu_parity import DELTA_TOL, mfbc, rel_close, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def graphs():
    gs = gg.batched_suite(count=5, seed0=7100, nmin=40, nmax=1200)
    gs.append(gg.star_graph(1500))
    gs.append(gg.csr_from_edges(3, [], [], None, "no_arcs"))
    gs.append(gg.path_graph(90, w=255))
    gs.append(gg.er_graph(300, 10, 7, (1, 6_000_000)))             # weights not packed
    return gs


@pytest.mark.parametrize("copies", [0, 150], ids=["few", "many"])
@pytest.mark.parametrize("plan", [{}, dict(run_arcs=4096, run_verts=64), dict(run_arcs=64, run_verts=5, heavy=30, slice=16)],
                         ids=["own", "coarse", "fine"])
def test_both_ways_against_the_oracle(torch, mfbc, copies, plan):  # noqa: F811
    gs = graphs()
    dgs = [mfbc.DeviceGraph(g) for g in gs]
    for d in dgs:
        if plan:
            d.set_plan(**plan)
    srcs = [np.arange(g.n, dtype=np.int32) for g in gs]
    srcs[0] = srcs[0][::3].copy()
    srcs[1] = srcs[1][:70].copy()
    gs.append(gs[2])                                                # the same handle again
    dgs.append(dgs[2])
    srcs.append(srcs[2][5:40].copy())
    gs.append(gs[3])
    dgs.append(dgs[3])
    srcs.append(np.zeros(0, dtype=np.int32))
    tiny = gg.er_graph(12, 3, 1, (1, 5))
    small = [mfbc.DeviceGraph(tiny) for _ in range(copies)]
    dgs[3].bc(np.arange(5, dtype=np.int32), 64)
    before = dgs[3].stats()
    want = [oracle.brandes(g, s, per_source=False)["lambda"] if s.size else np.zeros(g.n) for g, s in zip(gs, srcs)]
    first = None
    for width in (64, 128, 64):
        print(f"[batched] graphs={len(dgs) + copies} plan={plan} width={width}", flush=True)
        out = mfbc.bc_many(dgs + small, srcs + [np.arange(12, dtype=np.int32)] * copies, job_width=width)
        for g, w, o in zip(gs, want, out):
            rel_close(o.cpu().numpy(), w, DELTA_TOL, g.name)
        if width == 64:
            if first is not None:
                assert all(torch.equal(a, b) for a, b in zip(first, out)), "repeated calls are bitwise the same"
            first = out
        assert mfbc.bc_many.last_stats["fwd_products"] > 0
    assert dgs[3].stats() == before
    with pytest.raises(mfbc.MfbcError):
        mfbc.bc_many(dgs[:2], [srcs[0], np.array([10**6], dtype=np.int32)])
    for d in set(dgs) | set(small):
        d.close()
