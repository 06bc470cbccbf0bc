"""The library's host code on the CPU (csrc/mfbc_api.cpp built with g++ over
stand-ins for the HIP runtime and the kernel launchers, host/api_host.cpp):
what a call leaves behind when an allocation fails on its way.  At every
launch the stand-ins check that the plan and the workspace handed to the
kernel hold what it reads and writes, so a kernel that would read or write
out of range shows here and needs no GPU."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_1609_07008_amd import graphgen as gg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1609_07008_amd", "csrc")
HOST = os.path.join(ROOT, "tests", "host")
OK, EINVAL, ENOMEM, EDEVICE = 0, -1, -2, -3
P, I32, I64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    so = str(tmp_path_factory.mktemp("api") / "libapi_host.so")
    subprocess.run([cxx, "-O1", "-g", "-std=c++17", "-fPIC", "-shared", "-pthread",
                    "-I", os.path.join(HOST, "hip_stub"), "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(HOST, "api_host.cpp"),
                    *[os.path.join(CSRC, f) for f in ("mfbc_api.cpp", "graph.cpp", "order.cpp")], "-o", so],
                   check=True)
    return so


@pytest.fixture()
def lib(built):
    return bind(built)


def bind(so):
    x = ctypes.CDLL(so)
    x.stub_live.restype = x.stub_peak.restype = ctypes.c_size_t
    x.stub_faults.restype = x.stub_log.restype = x.mfbc_last_error.restype = ctypes.c_char_p
    x.stub_fail_in.argtypes = [ctypes.c_long]
    x.stub_cap.argtypes = [ctypes.c_size_t]
    x.stub_watch.argtypes = [P]
    x.mfbc_load_graph.argtypes = [I32, I64, P, P, P, ctypes.c_uint32, P, P]
    x.mfbc_free_graph.argtypes = [P]
    x.mfbc_set_plan.argtypes = [P, I32, I32, I32, I32]
    x.mfbc_set_lanes.argtypes = [P, I32]
    x.mfbc_forward.argtypes = [P, P, I32, P, P, P, P]
    x.mfbc_backward.argtypes = [P, P, I32, P, P, P, P, P]
    x.mfbc_fixpoint.argtypes = [P, I32, P, I32, P, P, P]
    x.mfbc_bc.argtypes = [P, P, I64, I32, P, P]
    x.mfbc_bc_noalloc.argtypes = [P, P, I64, I32, P, P]
    x.mfbc_bc_many.argtypes = [I32, P, P, P, P, P, P, P]
    x.stub_fail_in(-1)
    x.stub_cap(1 << 62)
    x.stub_products(3, 3)
    x.stub_core(100)
    x.stub_quad_fit(1 << 20)
    x.stub_watch(None)
    x.stub_clear()
    return x


def load(lib, g, directed=False):
    rp, col = np.ascontiguousarray(g.row_ptr, np.int64), np.ascontiguousarray(g.col, np.int32)
    w = None if g.w is None else np.ascontiguousarray(g.w, np.int32)
    h = P()
    rc = lib.mfbc_load_graph(g.n, col.size, rp.ctypes.data, col.ctypes.data, None if w is None else w.ctypes.data,
                             2 if directed else 1, None, ctypes.byref(h))
    return rc, h


def sources(nb):
    return np.arange(nb, dtype=np.int32)


def every_call(lib, h, n, nb=130):
    """One call of each kind whose products run on this handle's plans."""
    src, one = sources(nb), ctypes.c_double(0)
    out = ctypes.byref(one)          # the stand-ins write no results
    rcs = [lib.mfbc_forward(h, src.ctypes.data, nb, out, out, None, None),
           lib.mfbc_backward(h, src.ctypes.data, nb, out, out, out, None, None),
           *[lib.mfbc_fixpoint(h, op, src.ctypes.data, nb, out, None, None) for op in range(4)],
           lib.mfbc_bc(h, src.ctypes.data, nb, nb, out, None)]
    return rcs


KINDS = {
    "weighted": (lambda: gg.rmat_graph(9, 16, 3, wrange=(1, 255)), False, 40),       # with a core
    "unweighted": (lambda: gg.rmat_graph(9, 16, 3), False, 100),
    "directed": (lambda: gg.directed_rmat_graph(9, 16, 3, wrange=(1, 255)), True, 40),
}


@pytest.mark.parametrize("kind", list(KINDS))
def test_a_failed_set_plan_leaves_the_graph_as_it_was(lib, kind):
    """Every allocation of mfbc_set_plan in turn fails: ENOMEM, nothing leaked,
    and every call on the handle still finds whole plans and a workspace that
    holds their split rows; then the change goes through."""
    make, directed, percent = KINDS[kind]
    g = make()
    lib.stub_core(percent)
    before = lib.stub_live()
    rc, h = load(lib, g, directed)
    assert rc == OK
    for earlier in ((0, 0, 0, 0), (64, 5, 64, 32)):         # the library's own plans, then a caller's
        if any(earlier):
            assert lib.mfbc_set_plan(h, *earlier) == OK
        assert every_call(lib, h, g.n) == [OK] * 7
        held = lib.stub_live()
        failed = 0
        while True:
            lib.stub_fail_in(failed)
            rc = lib.mfbc_set_plan(h, 64, 3, 8, 2)          # many more slices than before
            lib.stub_fail_in(-1)
            if rc == OK:
                break
            assert rc == ENOMEM
            assert lib.stub_live() == held, f"allocation {failed}"
            assert every_call(lib, h, g.n) == [OK] * 7, f"allocation {failed}"
            assert lib.stub_faults() == b"", f"allocation {failed}"
            failed += 1
        assert failed >= (3 if percent == 100 else 6)
        assert every_call(lib, h, g.n) == [OK] * 7
    assert lib.mfbc_set_plan(h, 0, 0, 0, 0) == OK
    assert every_call(lib, h, g.n) == [OK] * 7
    assert lib.stub_faults() == b""
    lib.mfbc_free_graph(h)
    assert lib.stub_live() == before and lib.stub_faults() == b""


def ring(n, half=4):
    """Every vertex next to the `half` vertices on either side."""
    u = np.repeat(np.arange(n), half)
    return gg.csr_from_edges(n, u, (u + np.tile(np.arange(1, half + 1), n)) % n, None, f"ring{n}")


def admitted(n, arcs, groups):
    """The bytes that mfbc_bc_noalloc admits calls by (no row of these graphs
    is split): 39 B a (column, vertex) or so, 8 B a (group, arc)."""
    tile, nw = n * 64 * groups, (n + 31) // 32
    sizes = [4 * tile, 8 * tile, *2 * [4 * tile, 8 * tile, 8 * n * groups, 4 * nw * groups], 4, 8, 16384, 16,
             8 * n * groups, 8 * arcs * groups, 256 * groups, 2 * tile if groups > 1 else 4]
    return sum(-(-x // 256) * 256 for x in sizes) <= 64 << 20


@pytest.mark.parametrize("groups", [1, 2, 4])
def test_noalloc_admits_by_its_formula(lib, groups):
    """The largest ring that the formula admits runs, the next one is refused."""
    n = 28_100 // groups
    while not admitted(n, 8 * n, groups):
        n -= 1
    for n, want in ((n, OK), (n + 1, ENOMEM)):
        rc, h = load(lib, ring(n))
        assert rc == OK
        src, out = sources(64 * groups), ctypes.byref(ctypes.c_double(0))
        assert lib.mfbc_bc_noalloc(h, src.ctypes.data, src.size, src.size, out, None) == want, n
        lib.mfbc_free_graph(h)
    assert lib.stub_faults() == b""


def many(lib, graphs, nb, config=None):
    """mfbc_bc_many over loaded graphs, nb sources each; config: block_threads,
    blocks, job_width."""
    k = len(graphs)
    src, out = sources(nb), ctypes.c_double(0)
    cfg = np.array(config, np.int32) if config else None
    return lib.mfbc_bc_many(k, (P * k)(*graphs), (P * k)(*[src.ctypes.data] * k), (I64 * k)(*[nb] * k),
                            (P * k)(*[ctypes.addressof(out)] * k), cfg.ctypes.data if config else None, None, None)


@pytest.mark.parametrize("kind", list(KINDS))
def test_batched_form_on_streams_only_reads_the_handles(lib, kind):
    """A server may step on a graph while another thread has it in a batched
    call: the handle's plans and workspace stay what they are throughout."""
    make, directed, percent = KINDS[kind]
    lib.stub_core(percent)
    hs = [load(lib, make(), directed)[1] for _ in range(3)]
    assert every_call(lib, hs[0], 0) == [OK] * 7
    for plan in (None, (256, 64, 64, 32)):
        if plan:
            assert lib.mfbc_set_plan(hs[0], *plan) == OK
        lib.stub_watch(hs[0])
        assert many(lib, hs + hs[:1], 200) == OK         # (one graph listed twice)
        assert b"quad_product" in lib.stub_log() and b"bc_many" not in lib.stub_log()
        assert lib.stub_faults() == b""
        lib.stub_watch(None)
        lib.stub_clear()
    assert every_call(lib, hs[0], 0) == [OK] * 7
    for h in hs:
        lib.mfbc_free_graph(h)


def test_a_limit_on_the_workgroups_is_kept(lib):
    """Fewer workgroups than fill the device (2048 threads on each of 256 CUs)
    ask for the persistent launch on that many; else few graphs run on streams."""
    hs = [load(lib, KINDS["unweighted"][0]())[1] for _ in range(3)]
    for config, blocks in (((512, 37, 64), 37), ((256, 2047, 128), 2047), ((512, 1023, 0), 1023)):
        lib.stub_clear()
        assert many(lib, hs, 200, config) == OK
        assert lib.stub_log() == b"bc_many(%d) " % blocks
    for config in (None, (512, 1024, 128), (256, 2048, 64), (512, 0, 64)):
        lib.stub_clear()
        assert many(lib, hs, 200, config) == OK
        assert b"bc_many" not in lib.stub_log()
    for h in hs:
        lib.mfbc_free_graph(h)


def test_the_tuner_times_the_persistent_launch_alone(monkeypatch):
    """tune_many's launch shapes and plans shape the persistent launch only: every
    timed call asks for it, whatever its graphs."""
    import types

    import torch

    from paper_1609_07008_amd import autotune, mfbc
    calls = []
    empty = torch.empty
    monkeypatch.setattr(torch, "empty", lambda *a, device=None, **k: empty(*a, **k))
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda *a: types.SimpleNamespace(multi_processor_count=256))
    monkeypatch.setattr(mfbc, "bc_many", lambda *a, outs=None, **cfg: calls.append(cfg))
    graphs = [types.SimpleNamespace(n=n, set_plan=lambda **k: None) for n in (300, 3000, 9000)]
    cache = {}
    autotune.tune_many(graphs, [None] * 3, cache=cache)
    assert len(calls) > 20 and all(c["blocks"] * c["block_threads"] < 2048 * 256 for c in calls)
    assert cache["many"]["per_cu"] * cache["many"]["block_threads"] <= 2048      # the shape itself is kept


def test_default_lanes_take_what_fits(lib):
    """Where batches run at once by default, a lane whose workspace does not fit
    is left out; a lane count that was asked for is met or refused."""
    g = ring(1 << 15, 16)                                   # 2^20 arcs: four lanes at four groups
    src, out = sources(800), ctypes.byref(ctypes.c_double(0))
    lane, before = 0, lib.stub_live()
    for fit in (4, 0, 1, 2, 3):
        rc, h = load(lib, g)
        assert rc == OK
        start = lib.stub_live()
        lib.stub_cap(start + (2 * fit + 1) * lane // 2 if lane else 1 << 62)
        want = OK if fit else ENOMEM
        assert [lib.mfbc_bc(h, src.ctypes.data, src.size, 200, out, None) for _ in range(2)] == [want] * 2, fit
        held = lib.stub_live() - start
        lane = lane or held // 4
        assert held == fit * lane
        if fit < 4:
            assert lib.mfbc_set_lanes(h, 4) == OK
            assert lib.mfbc_bc(h, src.ctypes.data, src.size, 200, out, None) == ENOMEM
        lib.stub_cap(1 << 62)
        lib.mfbc_free_graph(h)
        assert lib.stub_live() == before and lib.stub_faults() == b""


@pytest.mark.parametrize("edges", [1 << 20, 1 << 16])
def test_default_lanes_stay_within_their_share(lib, edges):
    """n = 2^20 in batches of 448 columns (21 GB a batch): two at once on streams
    or, where arcs are few, in one wide batch; not four."""
    n, batch = 1 << 20, 448
    u = np.arange(edges)
    rc, h = load(lib, gg.csr_from_edges(n, u, (u + 1) % n, None, "path"))
    assert rc == OK
    src, out = sources(4 * batch), ctypes.byref(ctypes.c_double(0))
    lib.stub_reset_peak()
    assert lib.mfbc_bc(h, src.ctypes.data, src.size, batch, out, None) == OK
    assert round(lib.stub_peak() / (39 * n * 512)) == 2     # 39 B a (column, vertex), eight groups
    lib.mfbc_free_graph(h)
    assert lib.stub_faults() == b""


NO_THREADS = """
import resource, sys
sys.path.insert(0, {root!r})
from tests.test_host_api import *
lib = bind({so!r})
h = load(lib, ring(1 << 15, 16))[1]
hs = [load(lib, ring(2000, 4))[1] for _ in range(3)]
src, out = sources(800), ctypes.byref(ctypes.c_double(0))
resource.setrlimit(resource.RLIMIT_AS, (24 << 30, 24 << 30))
print(lib.mfbc_bc(h, src.ctypes.data, src.size, 200, out, None), many(lib, hs, 200),
      lib.stub_log().count(b"bwd_count"), lib.stub_faults())
"""


def test_lanes_whose_threads_cannot_start_run_all_the_same(built):
    """A process that cannot start a thread (stacks of 32 GiB within 24 GiB of
    address space): four batches and three graphs one after another, no abort."""
    import resource
    import sys
    hard = resource.getrlimit(resource.RLIMIT_STACK)[1]
    if hard not in (-1, resource.RLIM_INFINITY) and hard < 32 << 30:
        pytest.skip("stack sizes are limited here")
    r = subprocess.run([sys.executable, "-c", NO_THREADS.format(root=ROOT, so=built)], capture_output=True, text=True,
                       env=dict(os.environ, OPENBLAS_NUM_THREADS="1", OMP_NUM_THREADS="1"),
                       preexec_fn=lambda: resource.setrlimit(resource.RLIMIT_STACK, (32 << 30, hard)))
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split("\n")[-2] == "0 0 7 b''", r.stdout


@pytest.mark.parametrize("nb", [64, 384])
@pytest.mark.parametrize("percent", [100, 40])
def test_calls_without_room_for_16_bits_run_in_32(lib, nb, percent):
    """A device that holds the state of 32-bit products and not the 16-bit path
    counts or bounds beside it: the calls run, as they did before those."""
    lib.stub_core(percent)
    rc, h = load(lib, gg.rmat_graph(13, 32, 3, wrange=(1, 255)))          # more than 2^18 arcs
    src, out = sources(nb), ctypes.byref(ctypes.c_double(0))
    calls = {
        "forward": lambda: lib.mfbc_forward(h, src.ctypes.data, nb, out, out, None, None),
        "sssp": lambda: lib.mfbc_fixpoint(h, 0, src.ctypes.data, nb, out, None, None),
        "bc": lambda: lib.mfbc_bc(h, src.ctypes.data, nb, nb, out, None),
    }
    start = lib.stub_live()
    assert calls["bc"]() == OK and b"quad_product" in lib.stub_log()
    whole = lib.stub_live() - start
    # one word a lane less: none is left of one group's, three of six groups' four,
    # as many as the products on a core take
    least = whole - (1 << 13) * 64 * 4 + (4 if nb == 64 else 0)
    for cap, forms in ((whole, (False, False, True)), (least, (False, False, nb > 64)), (least - 4096, None)):
        for (name, call), form in zip(calls.items(), forms or (None,) * 3):
            lib.mfbc_free_graph(h)
            rc, h = load(lib, gg.rmat_graph(13, 32, 3, wrange=(1, 255)))
            lib.stub_clear()
            lib.stub_cap(lib.stub_live() + cap)
            assert call() == (ENOMEM if form is None else OK), (name, cap)
            assert (b"quad_product" in lib.stub_log()) == bool(form), (name, cap)
            lib.stub_cap(1 << 62)
    assert lib.stub_faults() == b""
    lib.mfbc_free_graph(h)


def test_products_that_ran_in_16_bits_are_not_run_again(lib):
    """A frontier that outlives the products whose entries fit (56 here): the
    call goes on in 32 bits from there, in every batch."""
    rc, h = load(lib, gg.rmat_graph(13, 32, 3, wrange=(1, 255)))          # more than 2^18 arcs
    lib.stub_quad_fit(56)
    src, out = sources(200), ctypes.byref(ctypes.c_double(0))
    count = ctypes.c_int32(0)
    for fwd in (56, 57, 100):
        lib.stub_products(fwd, 3)
        wide = 0 if fwd == 56 else -(-(fwd - 56) // 8) * 8
        for batches, name, call in (
                (1, b"fwd", lambda: lib.mfbc_forward(h, src.ctypes.data, 200, out, out, ctypes.byref(count), None)),
                (1, b"mono", lambda: lib.mfbc_fixpoint(h, 0, src.ctypes.data, 200, out, ctypes.byref(count), None)),
                (3, b"fwd", lambda: lib.mfbc_bc(h, src.ctypes.data, 200, 70, out, None))):
            lib.stub_clear()
            lib.mfbc_set_lanes(h, 1)
            assert call() == OK
            log = lib.stub_log()
            assert log.count(b"quad_product") == 56 * batches and log.count(name + b"_product") == wide * batches
            assert log.count(b"quad_widen") == (batches if wide else 0)
            assert count.value == fwd
    assert lib.stub_faults() == b""
    lib.mfbc_free_graph(h)


@pytest.mark.parametrize("scale,fit,kept", [(9, 56, False), (13, 56, True), (13, 0, False)])
def test_load_keeps_column_offsets_where_they_are_read(lib, scale, fit, kept):
    """The distances to one landmark serve the bounds of the 16-bit products on
    every arc: graphs of 2^18 arcs and more whose weights leave room for them."""
    lib.stub_quad_fit(fit)
    for percent in (40, 99):                                # with a core, and where one was tried
        lib.stub_core(percent)
        lib.stub_clear()
        rc, h = load(lib, gg.rmat_graph(scale, 32, 3, wrange=(1, 255)))
        assert rc == OK and (b"core_hub" in lib.stub_log()) == kept
        assert every_call(lib, h, 0) == [OK] * 7 and lib.stub_faults() == b""
        lib.mfbc_free_graph(h)
