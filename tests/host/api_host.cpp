// The library's host code (mfbc_api.cpp, graph.cpp, order.cpp) over stand-ins
// for the HIP runtime and the kernel launchers, so that its error paths can be
// run on the CPU: allocations that fail at a given point or beyond a given
// amount, and checks, at every launch, that the plan and the workspace handed
// to a kernel hold what that kernel reads and writes.  Built as a shared
// library and driven from test_host_api.py.
#include <sys/mman.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>

#include "mfbc_internal.h"

using namespace mfbc;

namespace {

constexpr size_t kMapped = (size_t)64 << 20;
std::mutex mu;
std::map<char *, size_t> blocks;         // live "device" allocations
size_t live = 0, peak = 0, cap = (size_t)1 << 62;
long fail_in = -1;                       // the allocation this many from now fails
std::string faults, log_;
int products = 3;                        // a frontier is empty from this product on
int core_percent = 100;                  // arcs kept in a core
int quad_fit = 1 << 20;                  // products that fit 16 bits
int bwd_products = 3;
const mfbc_graph *watched = nullptr;     // a handle that must not change while a call runs
Plan watched_out;
const void *watched_tdist = nullptr;

void fault(const std::string &what) {
    if (faults.size() < 4000) faults += what + "\n";
}

// Bytes from p to the end of the allocation it points into.
size_t room(const void *p) {
    if (!p) return 0;
    auto it = blocks.upper_bound((char *)p);
    if (it == blocks.begin()) return 0;
    --it;
    const size_t off = (size_t)((char *)p - it->first);
    return off < it->second ? it->second - off : 0;
}

void need(const char *who, const char *what, const void *p, size_t bytes) {
    if (bytes && room(p) < bytes)
        fault(std::string(who) + ": " + what + " holds " + std::to_string(room(p)) + " of " + std::to_string(bytes) +
              " bytes");
}

void check_plan(const char *who, const Plan &p, int64_t arcs) {
    if (p.ntasks < 1) fault(std::string(who) + ": no tasks");
    need(who, "tasks", p.tasks, (size_t)p.ntasks * sizeof(Task));
    need(who, "hubs", p.hubs, (size_t)p.nhubs * sizeof(Hub));
    need(who, "owner", p.owner, (size_t)arcs);
}

void check(const char *who, const mfbc_graph *g, const View &v, int ncg, bool quad) {
    std::lock_guard<std::mutex> lock(mu);
    if (log_.size() < 100000) log_ += std::string(who) + " ";
    check_plan(who, v.plan_in, v.arcs);
    check_plan(who, v.plan_out, v.arcs);
    const Workspace &ws = g->ws;
    const size_t tile = (size_t)g->n * kWave * (size_t)ncg;
    const size_t slots = (size_t)std::max(v.plan_in.nslots, v.plan_out.nslots) * kWave * (size_t)ncg;
    if (!ws.external) {
        need(who, "pd", ws.pd, slots * 4);
        need(who, "pm", ws.pm, slots * 8);
        need(who, "tdist", ws.tdist, tile * 4);
        need(who, "tsig", ws.tsig, tile * 8);
        need(who, "dag", ws.dag, v.arcs <= g->core.arcs ? (size_t)v.arcs * ncg * 8 : 0);
        if (quad)
            need(who, "tau2", ws.tau2,
                 (size_t)g->n * kWave * 4 * (size_t)((ncg + 2 * ws.quad.words - 1) / (2 * ws.quad.words)) * ws.quad.words);
    }
    if (watched && (watched->core.plan_out.tasks != watched_out.tasks ||
                    watched->core.plan_out.nslots != watched_out.nslots || watched->ws.tdist != watched_tdist))
        fault(std::string(who) + ": the handle's plan or workspace was exchanged");
}

void produced(mfbc_graph *g, int j, bool any) {
    unsigned long long *c = g->ws.counters + (size_t)(j % kCounterRing) * 4 * kCounterSlots;
    memset(c, 0, 4 * kCounterSlots * sizeof(*c));
    c[0] = any;
}

}  // namespace

extern "C" {
void stub_fail_in(long k) { fail_in = k; }
void stub_cap(size_t bytes) { cap = bytes; }
size_t stub_live() { return live; }
size_t stub_peak() { return peak; }
void stub_reset_peak() { peak = live; }
void stub_products(int fwd, int bwd) {
    products = fwd;
    bwd_products = bwd;
}
void stub_core(int percent) { core_percent = percent; }
void stub_quad_fit(int n) { quad_fit = n; }
void stub_watch(const mfbc_graph *g) {
    watched = g;
    if (!g) return;
    watched_out = g->core.plan_out;
    watched_tdist = g->ws.tdist;
}
const char *stub_faults() { return faults.c_str(); }
const char *stub_log() { return log_.c_str(); }
void stub_clear() {
    faults.clear();
    log_.clear();
}
}

// ------------------------------------------------------------------ runtime
const char *hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t bytes) {
    std::lock_guard<std::mutex> lock(mu);
    *p = nullptr;
    if (fail_in >= 0 && fail_in-- == 0) return hipErrorOutOfMemory;
    if (live + bytes > cap) return hipErrorOutOfMemory;
    // large blocks are never touched in full: address space alone
    if (bytes >= kMapped) {
        *p = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
        if (*p == MAP_FAILED) *p = nullptr;
    } else {
        *p = calloc(1, bytes ? bytes : 1);
    }
    if (!*p) return hipErrorOutOfMemory;
    blocks[(char *)*p] = bytes;
    live += bytes;
    peak = std::max(peak, live);
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    std::lock_guard<std::mutex> lock(mu);
    auto it = blocks.find((char *)p);
    if (it == blocks.end()) {
        fault("free of a pointer that is not live");
        return hipSuccess;
    }
    live -= it->second;
    if (it->second >= kMapped) munmap(p, it->second);
    else free(p);
    blocks.erase(it);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) {
    *p = calloc(1, bytes);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    free(p);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *f, size_t *t) {
    *t = std::min<size_t>(cap, (size_t)288 << 30);
    *f = *t > live ? *t - live : 0;
    return hipSuccess;
}
hipError_t hipMemcpy(void *to, const void *from, size_t bytes, hipMemcpyKind) {
    memcpy(to, from, bytes);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *to, const void *from, size_t bytes, hipMemcpyKind k, hipStream_t) {
    return hipMemcpy(to, from, bytes, k);
}
hipError_t hipMemsetAsync(void *p, int value, size_t bytes, hipStream_t) {
    memset(p, value, bytes);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *symbol) {
    *p = (void *)symbol;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *value, hipDeviceAttribute_t, int) {
    *value = 256;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = (hipStream_t)malloc(1);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    free(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) {
    *e = (hipEvent_t)malloc(1);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
    free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 0.f;
    return hipSuccess;
}

// ------------------------------------------------------------------ launchers
namespace mfbc {

void launch_fwd_init(mfbc_graph *g, int, int, const int32_t *, hipStream_t) { memset(g->ws.counters, 0, kCounterWords * 8); }
void launch_fwd_product(mfbc_graph *g, const View &v, int ncg, int j, hipStream_t, hipEvent_t *) {
    check("fwd_product", g, v, ncg, false);
    produced(g, j, j < products);
}
hipError_t launch_bwd_count(mfbc_graph *g, const View &v, int ncg, bool tau16, hipStream_t, hipEvent_t *) {
    check("bwd_count", g, v, ncg, tau16);
    produced(g, 0, true);
    return hipSuccess;
}
void launch_bwd_product(mfbc_graph *g, const View &v, int ncg, bool tau16, int k, hipStream_t, hipEvent_t *) {
    check("bwd_product", g, v, ncg, tau16);
    produced(g, k, k < bwd_products);
}
void launch_trace_fwd(mfbc_graph *, int, int, int, uint64_t *, hipStream_t) {}
void launch_set_sources_spans(mfbc_graph *, int, const int32_t *, const GroupSpans &, hipStream_t) {}
void launch_lambda_add_groups(mfbc_graph *, int, const GroupOuts &, hipStream_t) {}
void launch_zero_f64(double *, size_t, hipStream_t) {}
void launch_lambda_zero(mfbc_graph *g, int ncg, hipStream_t) {
    std::lock_guard<std::mutex> lock(mu);
    if (!g->ws.external) need("lambda_zero", "lam", g->ws.lam, (size_t)g->n * ncg * 8);
}
void launch_lambda_reduce(mfbc_graph *, int, double *, hipStream_t) {}
void launch_lambda_reduce_lanes(mfbc_graph *const *, int, int, double *, hipStream_t) {}
void launch_export_forward(mfbc_graph *, int, int, int32_t *, double *, hipStream_t) {}
void launch_import_forward(mfbc_graph *, int, int, const int32_t *, const double *, hipStream_t) {}
void launch_export_backward(mfbc_graph *, int, int, double *, int32_t *, hipStream_t) {}
void launch_set_sources(mfbc_graph *g, int, int, const int32_t *, hipStream_t) { g->ws.flags[2] = 0; }
void launch_check_sources(const int32_t *, int64_t, int, int32_t *bad, hipStream_t) { *bad = 0; }
void launch_export_tiles_i32(mfbc_graph *, int, int, const int32_t *, int32_t *, hipStream_t) {}

bool mono_op_known(int op) { return op >= 0 && op <= 3; }
void launch_mono_init(mfbc_graph *g, int, int, int, const int32_t *, hipStream_t) { memset(g->ws.counters, 0, kRingWords * 8); }
void launch_mono_product(mfbc_graph *g, int, int ncg, int j, hipStream_t, hipEvent_t *) {
    if (g->ws.tsig) check("mono_product", g, g->full, ncg, false);
    produced(g, j, j < products);
}

struct ManyWorkspace {
    char *scratch = nullptr;
    size_t bytes = 0;
};
ManyWorkspace &many_workspace(int) {
    static ManyWorkspace ws;
    return ws;
}
size_t many_slot_bytes(int, int, int64_t, int) { return 1 << 20; }
int launch_bc_many(std::vector<mfbc_graph *> &gs, const std::vector<const int32_t *> &, const std::vector<int64_t> &,
                   const std::vector<double *> &, int, int blocks, int, hipStream_t, ManyWorkspace &,
                   unsigned long long *st, int32_t *, std::string &) {
    std::lock_guard<std::mutex> lock(mu);
    log_ += "bc_many(" + std::to_string(blocks) + ") ";
    for (auto *g : gs) check_plan("bc_many", g->core.plan_out, g->core.arcs);
    st[0] = st[1] = gs.size();
    return MFBC_OK;
}
char *many_scratch(ManyWorkspace &ws, size_t bytes) {
    if (ws.bytes >= bytes) return ws.scratch;
    if (ws.scratch) (void)hipFree(ws.scratch);
    ws.bytes = 0;
    if (hipMalloc((void **)&ws.scratch, bytes) != hipSuccess) return nullptr;
    ws.bytes = bytes;
    return ws.scratch;
}
size_t ws_scratch_bytes_impl(const ManyWorkspace &ws) { return ws.bytes; }

bool bits_fit(const mfbc_graph *g, int op) { return op == MFBC_OP_BFS || g->maxw == 1; }
void launch_plan_owner(const Csr &, const Plan &pl, hipStream_t) {
    std::lock_guard<std::mutex> lock(mu);
    need("plan_owner", "tasks", pl.tasks, (size_t)pl.ntasks * sizeof(Task));
}
void launch_bits_init(mfbc_graph *g, int, int, const int32_t *, hipStream_t) { memset(g->ws.counters, 0, kRingWords * 8); }
void launch_bits_planes(mfbc_graph *, int, int, int, hipStream_t) {}
void launch_bits_product(mfbc_graph *g, int ncg, int j, hipStream_t, hipEvent_t *) {
    check("bits_product", g, g->full, ncg, false);
    produced(g, j, j < products);
}
void launch_bits_export(mfbc_graph *, int, int, int, int, void *, hipStream_t) {}

int quad_products(const mfbc_graph *, bool) { return quad_fit; }
size_t quad_bound_bytes(const mfbc_graph *g, int ncg, int, QuadBounds *, char *) { return (size_t)g->n * 10 * ncg; }
void launch_quad_init(mfbc_graph *g, const View &, bool, int, int, const int32_t *, hipStream_t) {
    memset(g->ws.counters, 0, kCounterWords * 8);
}
void launch_quad_product(mfbc_graph *g, const View &v, bool count, int ncg, int j, hipStream_t, hipEvent_t *) {
    check("quad_product", g, v, ncg, count);
    produced(g, j, j < products);
}
void launch_quad_widen(mfbc_graph *g, const View &v, bool count, int ncg, int, hipStream_t) {
    check("quad_widen", g, v, ncg, count);
}
void launch_quad_rows(mfbc_graph *, bool, int, int, int32_t *, double *, hipStream_t) {}

bool core_worth_trying(const mfbc_graph *g) { return g->weighted && core_percent < 100; }
bool sparse_rows(const mfbc_graph *) { return false; }
TaskParams core_params(int32_t n, int64_t arcs, int64_t) { return default_params(n, arcs); }
void launch_core_mark(const Csr &c, const Plan &, const int32_t *, const int32_t *, uint8_t *, int32_t *cnt, hipStream_t) {
    const size_t n = room(c.rp) / sizeof(int64_t) - 1;
    for (size_t v = 0; v < n; v++) cnt[v] = (int32_t)((c.rp[v + 1] - c.rp[v]) * core_percent / 100);
}
void launch_core_zero(int32_t *, int, hipStream_t) {}
void launch_core_hub(const int32_t *, int, int32_t *, hipStream_t) {
    std::lock_guard<std::mutex> lock(mu);
    log_ += "core_hub ";
}
void launch_core_compact(int32_t, const Csr &, const uint8_t *, const Csr &, hipStream_t) {}

}  // namespace mfbc
