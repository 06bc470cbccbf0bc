// C ABI of libmfbc (declared in include/mfbc.h): validation, device memory,
// and the host loops of Algorithms 1-3 around the HIP kernels.
//
// Per batch (Algorithm 3): initialise T and the first frontier (the sources
// themselves), then repeat the forward product until a product yields an
// empty frontier (Algorithm 1's loop condition, over all columns of the
// batch); then the counting product and the backward products until the
// backward frontier is empty (Algorithm 2); lambda parts are accumulated by
// the kernels as entries complete.  Products are enqueued in windows, and one
// copy per window brings back their frontier sizes and the error flags; that
// is the only host round trip of the loop.
#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstring>
#include <exception>
#include <functional>
#include <mutex>
#include <string>
#include <thread>
#include <type_traits>
#include <utility>
#include <vector>

#include "mfbc_internal.h"
#include "order.h"

using namespace mfbc;

// Scratch of mfbc_bc_noalloc: one file-scope device array per GPU (the code
// object's copy on each device), holding the workspace of one call.  Calls on
// one device share it; each call initialises what it reads.
// Calls are admitted by a fixed formula (ws_arrays) against kScratchBytes; the
// array is larger, since the default row cut of a small graph takes up to
// 4.7 MB more hub partials per group than the formula counts (rows cut into
// slices of max(64, arcs / 4096) arcs, 768 B each), a core's partials and
// DAG masks up to 1.4 B per arc more than the masks of every arc, path
// counts in 16 bits a tenth of a one-group workspace, and a third bitmap.
constexpr size_t kScratchBytes = (size_t)64 << 20;
constexpr size_t kScratchSize = (size_t)84 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchSize];

namespace {

thread_local std::string g_err;

int fail(int code, const std::string &msg) {
    g_err = msg;
    return code;
}

}  // namespace

int mfbc::set_error(int code, const std::string &msg) { return fail(code, msg); }

namespace {

#define HIP_TRY(expr)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess)                                                                \
            return fail(MFBC_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(e_));    \
    } while (0)

struct DeviceGuard {
    int prev = -1;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) == hipSuccess && prev != dev) (void)hipSetDevice(dev);
        else prev = -1;
    }
    ~DeviceGuard() {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};

template <typename T>
int dalloc(T **p, size_t count) {
    *p = nullptr;
    if (count == 0) count = 1;
    hipError_t e = hipMalloc((void **)p, count * sizeof(T));
    if (e != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();
        return fail(MFBC_ENOMEM, std::string("device allocation of ") +
                                     std::to_string(count * sizeof(T)) + " bytes failed");
    }
    return MFBC_OK;
}

template <typename T>
void dfree(T *&p) {
    if (p) (void)hipFree((void *)p);
    p = nullptr;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Every array of the per-batch workspace for `ncg` column groups, in a fixed
// order: f(pointer, element count).  Used both to allocate the arrays and to
// carve them out of one block of memory.
// (g == nullptr: every count is 0, for walks that need only the pointers.)
// tau_words: as Workspace::tau_words (ws_tau_words, unless that does not fit).
// admit: the sizes mfbc_bc_noalloc admits calls by -- the stored DAG of every
// arc, the hub partials of the plain row cut, two activity bitmaps -- which
// depend on neither the weights nor the default decomposition.
size_t ws_tau_words(int ncg, bool least) {
    if (least) return ncg >= 2 ? (size_t)ncg / 2 : 0;
    return ncg <= 2 ? 1 : 2 * (((size_t)ncg + 3) / 4);
}

template <typename F>
void ws_arrays(const mfbc_graph *g, Workspace &ws, int ncg, size_t tau_words, F &&f, bool admit = false) {
    const size_t n = g ? (size_t)g->n : 0;
    const size_t tile = n * kWave * (size_t)ncg;
    const size_t nwords = (n + 31) / 32;
    const size_t slots =
        g ? (size_t)(admit ? g->scratch_slots : max_slots(g)) * kWave * (size_t)ncg : 0;
    f(ws.tdist, tile);
    f(ws.tsig, tile);
    for (int b = 0; b < 2; b++) {
        f(ws.fdist[b], tile);
        f(ws.fsig[b], tile);
        f(ws.fbits[b], n * ncg);
    }
    for (int b = 0; b < (admit ? 2 : 3); b++) f(ws.abits[b], nwords * ncg);
    f(ws.pd, slots);
    f(ws.pm, slots);
    f(ws.counters, kCounterWords);
    f(ws.lam, n * ncg);
    f(ws.dag, (size_t)std::max<int64_t>(g ? (admit ? g->arcs : g->core.arcs) : 0, 1) * ncg);
    f(ws.src, (size_t)ncg * kWave);
    // the paired counting product's tau in 16 bits (`least`: what that takes), or
    // path counts in 16 bits (two words a lane from three groups on, as in quad.hip)
    f(ws.tau2, n * kWave * tau_words);
}

// Column groups the workspace holds for a batch of `ncg` groups: batches of
// two or more run the forward product on pairs, so their count is rounded up
// to whole pairs; a single group runs alone.
int ws_groups(int ncg) { return ncg <= 1 ? 1 : (ncg + 1) & ~1; }

// Bytes of the workspace of `ncg` groups when carved from one block.
size_t ws_bytes(const mfbc_graph *g, int ncg, bool admit) {
    Workspace tmp;
    size_t off = 0;
    ncg = ws_groups(ncg);
    ws_arrays(g, tmp, ncg, ws_tau_words(ncg, admit), [&](auto *&p, size_t count) {
        (void)p;
        off = align256(off + std::max<size_t>(count, 1) * sizeof(*p));
    }, admit);
    return off;
}

void free_workspace(Workspace &ws) {
    if (!ws.external) ws_arrays(nullptr, ws, 0, 0, [](auto *&p, size_t) { dfree(p); });
    dfree(ws.trace_relax);
    dfree(ws.quad_base);
    ws = Workspace{};
}

void free_plan(Plan &p) {
    dfree(p.tasks);
    dfree(p.hubs);
    dfree(p.owner);
    p.ntasks = p.nhubs = p.nslots = 0;
}

void free_csr(Csr &c) {
    dfree(c.rp);
    dfree(c.col);
    dfree(c.w);
    dfree(c.pk);
    c = Csr{};
}

// The plans of both orientations (of an undirected graph one plan, twice).
void free_plans(Plan &out, Plan &in) {
    if (in.tasks != out.tasks) free_plan(in);
    free_plan(out);
    in = Plan{};
}

// (an undirected view holds one orientation, twice)
void free_view(View &v) {
    free_plans(v.plan_out, v.plan_in);
    if (v.in.rp != v.out.rp) free_csr(v.in);
    free_csr(v.out);
    v = View{};
}

// Fills an empty plan; what it holds after a failure is the caller's to free.
int upload_plan(int32_t n, const int64_t *h_rp, const TaskParams &prm, Plan &plan) {
    std::vector<Task> tasks;
    std::vector<Hub> hubs;
    int32_t nslots = 0;
    build_plan(n, h_rp, prm, tasks, hubs, nslots);
    int rc;
    if ((rc = dalloc(&plan.tasks, tasks.size()))) return rc;
    if (!hubs.empty() && (rc = dalloc(&plan.hubs, hubs.size()))) return rc;
    if (!tasks.empty())
        HIP_TRY(hipMemcpy(plan.tasks, tasks.data(), tasks.size() * sizeof(Task), hipMemcpyHostToDevice));
    if (!hubs.empty())
        HIP_TRY(hipMemcpy(plan.hubs, hubs.data(), hubs.size() * sizeof(Hub), hipMemcpyHostToDevice));
    plan.ntasks = (int32_t)tasks.size();
    plan.nhubs = (int32_t)hubs.size();
    plan.nslots = nslots;
    return MFBC_OK;
}

// Grow the workspace to hold a batch of `ncg` column groups.  Where it does not
// fit with path counts in 16 bits, it holds the rest: such a batch runs in 32.
int ensure_workspace(mfbc_graph *g, int ncg) {
    Workspace &ws = g->ws;
    ncg = ws_groups(ncg);
    if (ws.ncg >= ncg && !ws.external) return MFBC_OK;
    free_workspace(ws);
    int rc = MFBC_OK;
    size_t tau = 0;
    for (bool least : {false, true}) {
        if (least && (rc != MFBC_ENOMEM || tau == ws_tau_words(ncg, true))) break;
        tau = ws_tau_words(ncg, least);
        rc = MFBC_OK;
        ws_arrays(g, ws, ncg, tau, [&](auto *&p, size_t count) {
            if (!rc) rc = dalloc(&p, count);
        });
        if (!rc) break;
        free_workspace(ws);
    }
    if (rc) return rc;
    ws.tau_words = (int)tau;
    ws.ncg = ncg;
    ws.flags = (int32_t *)(ws.counters + kRingWords);
    return MFBC_OK;
}

// Set up the workspace for 16-bit products with `words` 32-bit words per lane;
// with bounds (on every arc) the memory behind them is grown to the batch.
int ensure_quad(mfbc_graph *g, int ncg, int words, bool bounds) {
    Workspace &ws = g->ws;
    ws.quad = QuadBounds{};
    ws.quad.words = words;
    if (!bounds) return MFBC_OK;
    if (ws.quad_ncg < ncg) {
        dfree(ws.quad_base);
        ws.quad_ncg = 0;
        const int rc = dalloc(&ws.quad_base, quad_bound_bytes(g, ncg, 1, nullptr, nullptr));
        if (rc) return rc;
        ws.quad_ncg = ncg;
    }
    (void)quad_bound_bytes(g, ncg, words, &ws.quad, ws.quad_base);
    return MFBC_OK;
}

struct Counts {
    int64_t produced = 0, outputs = 0, active_vertices = 0, active_arcs = 0;
};

// Wait for the stream and copy the counter ring and the flags to the host.
int read_ring(mfbc_graph *g, hipStream_t s) {
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpyAsync(g->h_ctr, g->ws.counters, sizeof(unsigned long long) * kCounterWords,
                           hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    return MFBC_OK;
}

// Flag i of the workspace from the host copy.
int32_t ring_flag(const mfbc_graph *g, int i) { return ((const int32_t *)(g->h_ctr + kRingWords))[i]; }

// Counters of product `idx` from the host copy of the ring (see flush_counts).
Counts ring_counts(const mfbc_graph *g, int idx) {
    const size_t off = (size_t)(idx % kCounterRing) * 4 * kCounterSlots;
    int64_t t[4] = {0, 0, 0, 0};
    for (int k = 0; k < 4; k++)
        for (int i = 0; i < kCounterSlots; i++) t[k] += (int64_t)g->h_ctr[off + k * kCounterSlots + i];
    Counts c;
    c.produced = t[0];
    c.outputs = t[1];
    c.active_vertices = t[2];
    c.active_arcs = t[3];
    return c;
}

// Kernel times of the product launched in window position `i` (events
// recorded by the launchers).
// Kernel times of window position i: product kernel into *a, its merge into
// *b.  `fwd`: a forward or fixpoint product (timed in both timing modes).
void add_times(mfbc_graph *g, int i, double *a, double *b, bool fwd) {
    if (!g->timing || (g->timing == 2 && !fwd)) return;
    hipEvent_t *e = g->ev + 3 * i;
    float t0 = 0.f, t1 = 0.f;
    if (hipEventElapsedTime(&t0, e[0], e[1]) == hipSuccess) *a += t0;
    if (g->timing == 1 && hipEventElapsedTime(&t1, e[1], e[2]) == hipSuccess) *b += t1;
}

// Events for the launch at window position i (null: not timed).  Timing
// mode 2 records only the two around a forward or fixpoint product kernel:
// every event costs the stream a few microseconds, which small graphs'
// steps feel.
hipEvent_t *window_events(mfbc_graph *g, int i, bool fwd) {
    if (g->timing == 1) return g->ev + 3 * i;
    if (g->timing == 2 && fwd) return g->ev_pull + 3 * i;
    return nullptr;
}

int check_sources(mfbc_graph *g, const int32_t *d_sources, int64_t count, hipStream_t s) {
    if (count == 0) return MFBC_OK;
    if (!d_sources) return fail(MFBC_EINVAL, "sources pointer is NULL");
    std::vector<int32_t> h((size_t)count);
    HIP_TRY(hipMemcpyAsync(h.data(), d_sources, (size_t)count * sizeof(int32_t),
                           hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    for (int64_t i = 0; i < count; i++)
        if (h[(size_t)i] < 0 || h[(size_t)i] >= g->n)
            return fail(MFBC_EINVAL, "source " + std::to_string(h[(size_t)i]) + " at position " +
                                         std::to_string(i) + " is outside [0, n)");
    return MFBC_OK;
}

// A batch's sources are checked by the kernel that sets them; the flag comes
// back with the first window's counters, before any output is written.  The
// message names the source.
int bad_source(mfbc_graph *g, const int32_t *d_sources, int64_t count, hipStream_t s) {
    const int rc = check_sources(g, d_sources, count, s);
    return rc ? rc : fail(MFBC_EINVAL, "a source is outside [0, n)");
}

// Algorithm 1 on a batch of sources (d_sources nullable: already in ws.src).
//
// Products are enqueued kWindow at a time and their counters read back
// once per window: a product whose predecessor produced nothing skips
// itself on the device, so the products past the end of the loop in the
// last window cost a launch each and change nothing.  The loop ends at the
// first product that produced no frontier entry (Algorithm 1's condition
// over every column of the batch).
// Trace (d_rows non-null or h_relax non-null): frontier membership of F_j
// after every product j <= max_products, as vertex bitmaps per column
// (d_rows + (j-1) * nb * words), and the relaxations of every product.
// from: the products that ran in 16 bits (run_quad), whose state is in place.
struct Begun {
    int j = 0;               // products run
    int64_t prev = 0;        // entries of the last one's frontier
};

int run_forward(mfbc_graph *g, const View &vw, int ncg, int nb, const int32_t *d_sources, const Begun &from, bool trace,
                uint64_t *d_rows, int64_t *h_nnz, int64_t *h_relax, int max_products, int32_t *products,
                hipStream_t s) {
    if (!from.j) launch_fwd_init(g, ncg, nb, d_sources, s);
    if (trace) launch_trace_fwd(g, ncg, nb, 0, nullptr, s);
    const double arc_bytes = g->weighted ? 8.0 : 4.0;
    const size_t words = ((size_t)g->n + 63) / 64;
    mfbc_stats &st = g->stats;
    int64_t prev = from.j ? from.prev : nb;      // the first frontier: one entry per source column
    int j = from.j, last = 0;
    while (!last) {
        if (j > g->n + 1) return fail(MFBC_EDEVICE, "forward products did not converge");
        for (int i = 0; i < kWindow; i++) {
            const int jj = j + 1 + i;
            launch_fwd_product(g, vw, ncg, jj, s, window_events(g, i, true));
            if (trace)
                launch_trace_fwd(g, ncg, nb, jj,
                                 d_rows && jj <= max_products ? d_rows + (size_t)(jj - 1) * nb * words
                                                              : nullptr,
                                 s);
        }
        int rc = read_ring(g, s);
        if (rc) return rc;
        if (j == 0 && d_sources && ring_flag(g, 2)) return bad_source(g, d_sources, nb, s);
        for (int i = 0; i < kWindow; i++) {
            const int jj = j + 1 + i;
            st.fwd_pull_launches++;
            add_times(g, i, &st.fwd_pull_ms, &st.fwd_merge_ms, true);
            if (last) continue;          // skipped on the device
            const Counts c = ring_counts(g, jj);
            if (h_nnz && jj <= max_products) h_nnz[jj - 1] = c.produced;
            st.fwd_entries += c.produced;
            st.fwd_outputs += c.outputs;
            st.fwd_active_vertices += c.active_vertices;
            st.fwd_active_arcs += c.active_arcs;
            st.fwd_alg_bytes += 8.0 * c.active_vertices + arc_bytes * c.active_arcs +
                                12.0 * (double)(prev + c.outputs + c.produced);
            prev = c.produced;
            if (c.produced == 0) last = jj;
        }
        j += kWindow;
    }
    g->stats.fwd_products += last;
    if (products) *products = last;
    if (trace && h_relax) {
        const int k = std::min(last, max_products);
        std::vector<unsigned long long> r((size_t)k + 1, 0ull);
        HIP_TRY(hipMemcpyAsync(r.data(), g->ws.trace_relax, sizeof(unsigned long long) * ((size_t)k + 1),
                               hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        for (int i = 0; i < k; i++) h_relax[i] = (int64_t)r[(size_t)i];
    }
    if (ring_flag(g, 0)) return fail(MFBC_EOVERFLOW, "a shortest-path count overflowed binary64");
    return MFBC_OK;
}

// Below this many arcs mfbc_forward and the fixpoint stay in 32 bits: a task's
// fixed cost (bounds, live columns) shows there.  256 sources on weighted R-MAT
// graphs, ms in 32 / 16 bits: path counts at scale 12 0.85 / 0.95, 13 0.94 /
// 1.04, 14 1.53 / 1.40, 16 3.68 / 1.99, 18 (200 sources) 10.0 / 4.5; distances
// 0.67 / 0.69, 0.84 / 1.00, 1.28 / 1.22, 2.69 / 1.64, 6.6 / 2.5.
constexpr int64_t kQuadArcs = 1 << 18;

// Algorithm 1, or the (min, a + w) fixpoint without multiplicities, in 16 bits
// (d_sources nullable: already in ws.src): on every arc with bounds, on the
// core without.  *fits becomes false if the state has no room, or if the
// frontier outlives the products whose entries fit: then *begun says how many
// ran, and the state is left as the next product in 32 bits reads it.
int run_quad(mfbc_graph *g, bool core, bool count, int ncg, int nb, const int32_t *d_sources, int32_t *products,
             bool *fits, Begun *begun, hipStream_t s) {
    const View &vw = core ? g->core : g->full;
    const int words = core || ncg <= 2 ? 1 : 2;
    const int most = core || g->arcs >= kQuadArcs ? quad_products(g, count) : 0;
    *fits = most > 0 && (!count || (ncg + 2 * words - 1) / (2 * words) * words <= g->ws.tau_words);
    if (!*fits) return MFBC_OK;
    int rc = ensure_quad(g, ncg, words, !core);
    if (rc == MFBC_ENOMEM) {
        *fits = false;
        return MFBC_OK;
    }
    if (rc) return rc;
    launch_quad_init(g, vw, count, ncg, nb, d_sources, s);
    const double arc_bytes = g->weighted ? 8.0 : 4.0;
    mfbc_stats &st = g->stats;
    int64_t prev = nb;
    int j = 0, last = 0;
    while (!last) {
        if (j + kWindow > most) {
            *fits = false;
            launch_quad_widen(g, vw, count, ncg, j, s);
            begun->j = j;
            begun->prev = prev;
            return MFBC_OK;
        }
        for (int i = 0; i < kWindow; i++) launch_quad_product(g, vw, count, ncg, j + 1 + i, s, window_events(g, i, true));
        if ((rc = read_ring(g, s))) return rc;
        if (j == 0 && d_sources && ring_flag(g, 2)) return bad_source(g, d_sources, nb, s);
        for (int i = 0; i < kWindow; i++) {
            const int jj = j + 1 + i;
            st.fwd_pull_launches++;
            add_times(g, i, &st.fwd_pull_ms, &st.fwd_merge_ms, true);
            if (last) continue;
            const Counts c = ring_counts(g, jj);
            st.fwd_entries += c.produced;
            st.fwd_outputs += c.outputs;
            st.fwd_active_vertices += c.active_vertices;
            st.fwd_active_arcs += c.active_arcs;
            st.fwd_alg_bytes += 8.0 * c.active_vertices + arc_bytes * c.active_arcs +
                                (count ? 12.0 * (double)(prev + c.outputs + c.produced)
                                       : 4.0 * (double)(prev + c.outputs) + 8.0 * (double)c.produced);
            prev = c.produced;
            if (c.produced == 0) last = jj;
        }
        j += kWindow;
    }
    if (count && ring_flag(g, 0)) return fail(MFBC_EOVERFLOW, "a shortest-path count overflowed binary64");
    st.fwd_products += last;
    if (products) *products = last;
    return MFBC_OK;
}

// Algorithm 2 on the batch whose T is in the workspace: the counting
// product (window position 0 of the first window), then backward products
// in windows as in run_forward, until one produces no frontier entry.
int run_backward(mfbc_graph *g, const View &vw, int ncg, int nb, bool tau16, int32_t *products, hipStream_t s) {
    const double arc_bytes = g->weighted ? 8.0 : 4.0;
    mfbc_stats &st = g->stats;
    int64_t prev = 0;
    int k = 0, last = -1;
    while (last < 0) {
        if (k > g->n + 1) return fail(MFBC_EDEVICE, "backward products did not converge");
        for (int i = 0; i < kWindow; i++) {
            const int kk = k + i;
            if (kk == 0) {
                const hipError_t e = launch_bwd_count(g, vw, ncg, tau16, s, window_events(g, i, false));
                if (e != hipSuccess)
                    return fail(MFBC_EDEVICE, std::string("counting product: ") + hipGetErrorString(e));
            } else {
                launch_bwd_product(g, vw, ncg, tau16, kk, s, window_events(g, i, false));
            }
        }
        int rc = read_ring(g, s);
        if (rc) return rc;
        for (int i = 0; i < kWindow; i++) {
            const int kk = k + i;
            if (kk == 0) {
                const Counts c = ring_counts(g, 0);
                st.bwd_entries += c.produced;
                st.count_launches++;
                // adjacency, tau of every (column, vertex) read once, the
                // stored DAG (one 8-byte lane mask per arc and column group)
                // written, the backward state of every (column, vertex)
                // initialised (counter 4 B, zeta 8 B, frontier index 4 B
                // when traced), and each leaf's sigma read and 1/sigma written
                const double state = g->trace_step ? 16.0 : 12.0;
                st.count_alg_bytes += arc_bytes * (double)vw.arcs + 8.0 * g->n +
                                      (8.0 + state) * (double)g->n * nb +
                                      8.0 * (double)vw.arcs * ncg + 16.0 * (double)c.produced;
                if (g->timing == 1) {
                    float t = 0.f;
                    if (hipEventElapsedTime(&t, g->ev[0], g->ev[2]) == hipSuccess) st.count_ms += t;
                }
                prev = c.produced;
                if (c.produced == 0) last = 0;
                continue;
            }
            st.bwd_pull_launches++;
            add_times(g, i, &st.bwd_pull_ms, &st.bwd_merge_ms, false);
            if (last >= 0) continue;      // skipped on the device
            const Counts c = ring_counts(g, kk);
            st.bwd_entries += c.produced;
            st.bwd_outputs += c.outputs;
            st.bwd_active_vertices += c.active_vertices;
            st.bwd_active_arcs += c.active_arcs;
            // + the DAG lane mask of every arc with an active head (8 B)
            st.bwd_alg_bytes += 8.0 * c.active_vertices + (arc_bytes + 8.0) * c.active_arcs +
                                12.0 * (double)prev + 24.0 * (double)c.outputs;
            prev = c.produced;
            if (c.produced == 0) last = kk;
        }
        k += kWindow;
    }
    st.bwd_products += last + 1;
    if (products) *products = last + 1;
    return MFBC_OK;
}

// One batch of Algorithm 3: the forward products in 16 bits where they fit (two
// groups to a word, the layout that the counting product reads), else, or from
// the first one that does not, in 32.
int run_batch(mfbc_graph *g, int ncg, int nb, const int32_t *d_sources, hipStream_t s) {
    int rc;
    bool tau16 = false;
    Begun begun;
    if ((rc = run_quad(g, true, true, ncg, nb, d_sources, nullptr, &tau16, &begun, s))) return rc;
    if (!tau16 && (rc = run_forward(g, g->core, ncg, nb, d_sources, begun, false, nullptr, nullptr, nullptr, 0, nullptr,
                                    s)))
        return rc;
    return run_backward(g, g->core, ncg, nb, tau16, nullptr, s);
}

int forward_impl(mfbc_graph *g, const int32_t *d_sources, int32_t nb, int32_t *d_dist,
                 double *d_sigma, bool trace, uint64_t *d_rows, int64_t *h_nnz, int64_t *h_relax,
                 int32_t max_products, int32_t *h_products, void *stream) {
    if (!g) return fail(MFBC_EINVAL, "graph handle is NULL");
    if (nb < 1) return fail(MFBC_EINVAL, "nb must be >= 1");
    if (!d_dist || !d_sigma) return fail(MFBC_EINVAL, "output pointer is NULL");
    if (trace && max_products < 0) return fail(MFBC_EINVAL, "max_products must be >= 0");
    if (!d_sources) return fail(MFBC_EINVAL, "sources pointer is NULL");
    DeviceGuard dg(g->device);
    hipStream_t s = (hipStream_t)stream;
    int rc;
    const int ncg = (nb + kWave - 1) / kWave;
    if ((rc = ensure_workspace(g, ncg))) return rc;
    if (trace) {
        // the trace's buffers are outputs: the sources are checked before they are cleared
        if ((rc = check_sources(g, d_sources, nb, s))) return rc;
        // relaxations of products 1 .. n + 1 + kWindow (every product a loop can launch)
        const int need = g->n + 2 + kWindow;
        if (g->ws.trace_len < need) {
            dfree(g->ws.trace_relax);
            g->ws.trace_len = 0;
            if ((rc = dalloc(&g->ws.trace_relax, (size_t)need))) return rc;
            g->ws.trace_len = need;
        }
        HIP_TRY(hipMemsetAsync(g->ws.trace_relax, 0, sizeof(unsigned long long) * (size_t)need, s));
        if (d_rows && max_products > 0)
            HIP_TRY(hipMemsetAsync(d_rows, 0,
                                   sizeof(uint64_t) * (size_t)max_products * nb * (((size_t)g->n + 63) / 64),
                                   s));
    }
    g->stats = mfbc_stats{};
    bool fits = false;
    Begun begun;
    if (!trace && (rc = run_quad(g, false, true, ncg, nb, d_sources, h_products, &fits, &begun, s))) return rc;
    if (fits) {
        g->stats.batches = 1;
        launch_quad_rows(g, true, ncg, nb, d_dist, d_sigma, s);
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipStreamSynchronize(s));
        return MFBC_OK;
    }
    if ((rc = run_forward(g, g->full, ncg, nb, d_sources, begun, trace, d_rows, h_nnz, h_relax, max_products, h_products,
                          s)))
        return rc;
    g->stats.batches = 1;
    launch_export_forward(g, ncg, nb, d_dist, d_sigma, s);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(s));
    return MFBC_OK;
}

int backward_impl(mfbc_graph *g, const int32_t *d_sources, int32_t nb, const int32_t *d_dist,
                  const double *d_sigma, double *d_delta, int32_t *d_step, int32_t *h_products,
                  void *stream) {
    if (!g) return fail(MFBC_EINVAL, "graph handle is NULL");
    if (nb < 1) return fail(MFBC_EINVAL, "nb must be >= 1");
    if (!d_dist || !d_sigma || !d_delta) return fail(MFBC_EINVAL, "array pointer is NULL");
    if (!d_sources) return fail(MFBC_EINVAL, "sources pointer is NULL");
    DeviceGuard dg(g->device);
    hipStream_t s = (hipStream_t)stream;
    int rc;
    const int ncg = (nb + kWave - 1) / kWave;
    if ((rc = ensure_workspace(g, ncg))) return rc;
    g->stats = mfbc_stats{};
    launch_set_sources(g, ncg, nb, d_sources, s);
    launch_import_forward(g, ncg, nb, d_dist, d_sigma, s);
    g->trace_step = d_step != nullptr;
    int32_t products = 0;
    rc = run_backward(g, g->core, ncg, nb, false, &products, s);
    g->trace_step = false;
    if (rc) return rc;
    if (ring_flag(g, 2)) return bad_source(g, d_sources, nb, s);
    if (h_products) *h_products = products;
    g->stats.batches = 1;
    launch_export_backward(g, ncg, nb, d_delta, d_step, s);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(s));
    return MFBC_OK;
}

int bits_for(int64_t x) {
    int b = 0;
    while (x > 0) {
        b++;
        x >>= 1;
    }
    return b;
}

// Device copy of one CSR orientation; weighted rows also get the packed
// (column | weight << cb) words when both fit 32 bits, halving arc traffic.
int upload_csr(int32_t n, int64_t arcs, const int64_t *rp, const int32_t *col, const int32_t *w,
               int32_t maxw, Csr &c) {
    int rc;
    if ((rc = dalloc(&c.rp, (size_t)n + 1)) || (rc = dalloc(&c.col, (size_t)arcs))) return rc;
    HIP_TRY(hipMemcpy(c.rp, rp, ((size_t)n + 1) * sizeof(int64_t), hipMemcpyHostToDevice));
    if (arcs) HIP_TRY(hipMemcpy(c.col, col, (size_t)arcs * sizeof(int32_t), hipMemcpyHostToDevice));
    if (w) {
        if ((rc = dalloc(&c.w, (size_t)arcs))) return rc;
        if (arcs) HIP_TRY(hipMemcpy(c.w, w, (size_t)arcs * sizeof(int32_t), hipMemcpyHostToDevice));
        const int cb = std::max(1, bits_for((int64_t)n - 1));
        if (cb + bits_for(maxw) <= 32) {
            std::vector<uint32_t> pk((size_t)arcs);
            for (int64_t e = 0; e < arcs; e++)
                pk[(size_t)e] = (uint32_t)col[e] | ((uint32_t)w[e] << cb);
            if ((rc = dalloc(&c.pk, (size_t)arcs))) return rc;
            if (arcs)
                HIP_TRY(hipMemcpy(c.pk, pk.data(), (size_t)arcs * sizeof(uint32_t),
                                  hipMemcpyHostToDevice));
            c.cb = cb;
        }
    }
    return MFBC_OK;
}

// New plans for the arcs of one view (one for both orientations of an
// undirected graph); both stay empty on a failure.
int make_plans(int32_t n, bool directed, const std::vector<int64_t> &rp_out, const std::vector<int64_t> &rp_in,
               const TaskParams &p, const View &v, Plan &out, Plan &in) {
    auto fill = [&](const std::vector<int64_t> &rp, const Csr &csr, Plan &plan) {
        int rc = upload_plan(n, rp.data(), p, plan);
        if (!rc && !(rc = dalloc(&plan.owner, (size_t)rp.back()))) launch_plan_owner(csr, plan, nullptr);
        return rc;
    };
    int rc = fill(rp_out, v.out, out);
    if (!rc && directed) rc = fill(rp_in, v.in, in);
    if (!rc && (hipGetLastError() != hipSuccess || hipStreamSynchronize(nullptr) != hipSuccess))
        rc = fail(MFBC_EDEVICE, "the plan's row bytes could not be written");
    if (rc) free_plans(out, in);
    else if (!directed) in = out;
    return rc;
}

// Work decompositions of both views; knobs <= 0 take the default of the
// view's own size.  The plans in use are replaced once all new ones are
// there: a failure leaves the graph as it was.
int plan_views(mfbc_graph *g, const TaskParams &knobs) {
    auto params = [&](bool core) {
        TaskParams p = core ? core_params(g->n, g->core.arcs, g->full.arcs) : default_params(g->n, g->full.arcs);
        if (knobs.run_arcs > 0) p.run_arcs = knobs.run_arcs;
        if (knobs.run_verts > 0) p.run_verts = knobs.run_verts;
        if (knobs.heavy > 0) p.heavy = knobs.heavy;
        if (knobs.slice > 0) p.slice = knobs.slice;
        return p;
    };
    Plan out, in, core_out, core_in;
    int rc = make_plans(g->n, g->directed, g->h_rp_out, g->h_rp_in, params(false), g->full, out, in);
    if (!rc && g->has_core)
        rc = make_plans(g->n, g->directed, g->h_core_rp_out, g->h_core_rp_in, params(true), g->core, core_out, core_in);
    if (rc) {
        free_plans(out, in);
        return rc;
    }
    // the first plans of the products that run on the core (on every arc where
    // there is none) are the library's own and stay
    const bool keep = g->core.plan_out.tasks && !g->own_out.tasks;
    if (keep) {
        g->own_out = g->core.plan_out;
        g->own_in = g->core.plan_in;
    } else if (g->has_core) {
        free_plans(g->core.plan_out, g->core.plan_in);
    }
    if (g->has_core || !keep) free_plans(g->full.plan_out, g->full.plan_in);
    g->full.plan_out = out;
    g->full.plan_in = in;
    if (g->has_core) {
        g->core.plan_out = core_out;
        g->core.plan_in = core_in;
    } else {
        g->core = g->full;
    }
    g->params = params(false);
    // slots of a decomposition with the plain row cut (or the caller's): what
    // mfbc_bc_noalloc counts, whatever the default cut is
    const int64_t heavy = knobs.heavy > 0 ? knobs.heavy : kPlainHeavy;
    const int64_t slice = knobs.slice > 0 ? knobs.slice : kPlainSlice;
    g->scratch_slots = 0;
    for (const auto *rp : {&g->h_rp_out, &g->h_rp_in}) {
        int64_t t = 0;
        for (int32_t v = 0; v < g->n; v++) {
            const int64_t d = (*rp)[(size_t)v + 1] - (*rp)[(size_t)v];
            if (d > heavy) t += (d + slice - 1) / slice;
        }
        g->scratch_slots = std::max(g->scratch_slots, t);
        if (!g->directed) break;
    }
    return MFBC_OK;
}

// One block of device memory, handed out in parts and freed at the end of
// the scope: take() before alloc() adds up the sizes, after it places them.
struct Scratch {
    char *base = nullptr;
    size_t off = 0;
    template <typename T>
    void take(T **p, size_t count) {
        *p = base ? (T *)(base + off) : nullptr;
        off = align256(off + std::max<size_t>(count, 1) * sizeof(T));
    }
    bool alloc() {
        const size_t need = off;
        off = 0;
        if (hipMalloc((void **)&base, need) == hipSuccess) return true;
        (void)hipGetLastError();
        base = nullptr;
        return false;
    }
    ~Scratch() {
        if (base) (void)hipFree(base);
    }
};

// Upper bounds of the distances from the landmarks (ws.src) to every vertex
// along the arcs of t.full.in, in t.ws.tdist: the walks of at most six
// arcs.  Longer ones drop few arcs more (arcs kept by walks of up to 6 / any:
// uniform graphs of degree 256 7.1% / 6.9%, of degree 40 33% / 31%; R-MAT
// scale 16 8.7% / 8.7%).
void landmark_bounds(mfbc_graph &t, int count, hipStream_t s) {
    launch_mono_init(&t, MFBC_OP_SSSP, 1, count, nullptr, s);
    for (int j = 1; j <= 6; j++) launch_mono_product(&t, MFBC_OP_SSSP, 1, j, s, nullptr);
}

// The core of one orientation: rows of bounds `near` for the row vertices,
// `far` for the others.  Leaves c2 empty if too few arcs go.
int core_csr(mfbc_graph *g, const Csr &c, const Plan &pl, const int32_t *near, const int32_t *far,
             uint8_t *keep, int32_t *cnt, Csr &c2, std::vector<int64_t> &rp2, hipStream_t s) {
    std::vector<int32_t> h((size_t)g->n);
    launch_core_zero(cnt, g->n, s);
    launch_core_mark(c, pl, near, far, keep, cnt, s);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpyAsync(h.data(), cnt, (size_t)g->n * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    rp2.resize((size_t)g->n + 1);
    rp2[0] = 0;
    for (int32_t v = 0; v < g->n; v++) rp2[(size_t)v + 1] = rp2[(size_t)v] + h[(size_t)v];
    const int64_t arcs = rp2.back();
    // a core of nearly every arc saves little and costs its memory
    if ((double)arcs > 0.75 * (double)g->arcs) return MFBC_OK;
    int rc;
    // packed arcs are all that the products read
    if ((rc = dalloc(&c2.rp, rp2.size())) || (c.pk && (rc = dalloc(&c2.pk, (size_t)arcs))) ||
        (!c.pk && ((rc = dalloc(&c2.col, (size_t)arcs)) || (rc = dalloc(&c2.w, (size_t)arcs)))))
        return rc;
    c2.cb = c.cb;
    HIP_TRY(hipMemcpyAsync(c2.rp, rp2.data(), rp2.size() * sizeof(int64_t), hipMemcpyHostToDevice, s));
    launch_core_compact(g->n, c, keep, c2, s);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(s));
    return MFBC_OK;
}

// Builds g->core (core.hip).  The graph stays without one where memory for
// the bounds is short or too few arcs go; both are no error.
int build_core(mfbc_graph *g, hipStream_t s) {
    const size_t n = (size_t)g->n, tile = n * kWave;
    // landmarks: the vertices of highest degree
    const int count = (int)std::min<size_t>(n, (size_t)kLandmarks);
    std::vector<int32_t> v(n);
    for (size_t i = 0; i < n; i++) v[i] = (int32_t)i;
    auto deg = [&](int32_t x) {
        return g->h_rp_out[(size_t)x + 1] - g->h_rp_out[(size_t)x] + g->h_rp_in[(size_t)x + 1] -
               g->h_rp_in[(size_t)x];
    };
    if (g->h_perm.empty())     // else the numbering is by descending degree already
        std::partial_sort(v.begin(), v.begin() + count, v.end(), [&](int32_t a, int32_t b) {
            return deg(a) != deg(b) ? deg(a) > deg(b) : a < b;
        });
    Scratch mem;
    mfbc_graph t;
    t.device = g->device;
    t.n = g->n;
    t.arcs = g->arcs;
    t.maxw = g->maxw;
    t.weighted = true;
    t.full = g->full;
    Workspace &ws = t.ws;
    const size_t words = (n + 31) / 32;
    int32_t *from = nullptr, *to = nullptr, *cnt = nullptr;
    uint8_t *keep = nullptr;
    for (int pass = 0; pass < 2; pass++) {
        mem.take(&from, tile);
        if (g->directed) mem.take(&to, tile);
        for (int i = 0; i < 2; i++) {
            mem.take(&ws.fdist[i], tile);
        }
        for (auto &b : ws.abits) mem.take(&b, words);
        mem.take(&ws.pd, (size_t)max_slots(g) * kWave);
        mem.take(&ws.counters, kCounterWords);
        mem.take(&ws.src, (size_t)kWave);
        mem.take(&keep, (size_t)g->arcs);
        mem.take(&cnt, n);
        if (pass == 0 && !mem.alloc()) return MFBC_OK;
    }
    HIP_TRY(hipMemcpyAsync(ws.src, v.data(), (size_t)count * sizeof(int32_t), hipMemcpyHostToDevice, s));
    int rc;
    ws.tdist = from;
    landmark_bounds(t, count, s);
    if (g->directed) {
        std::swap(t.full.in, t.full.out);
        std::swap(t.full.plan_in, t.full.plan_out);
        ws.tdist = to;
        landmark_bounds(t, count, s);
    } else {
        to = from;
    }
    // kept as the columns' offsets in the bounds of quad.hip, core or not
    const bool bounds = g->arcs >= kQuadArcs && (quad_products(g, true) > 0 || quad_products(g, false) > 0);
    if (bounds && !dalloc(&g->hub_dist, n)) launch_core_hub(to, g->n, g->hub_dist, s);
    View c;
    rc = core_csr(g, g->full.out, g->full.plan_out, to, from, keep, cnt, c.out, g->h_core_rp_out, s);
    if (!rc && c.out.rp && g->directed)
        rc = core_csr(g, g->full.in, g->full.plan_in, from, to, keep, cnt, c.in, g->h_core_rp_in, s);
    if (rc || !c.out.rp) {
        free_view(c);
        return rc == MFBC_ENOMEM ? MFBC_OK : rc;
    }
    if (!g->directed) {
        c.in = c.out;
        g->h_core_rp_in = g->h_core_rp_out;
    }
    c.arcs = g->h_core_rp_out.back();
    rc = make_plans(g->n, g->directed, g->h_core_rp_out, g->h_core_rp_in, core_params(g->n, c.arcs, g->full.arcs), c,
                    c.plan_out, c.plan_in);
    if (rc) {
        free_view(c);
        return rc == MFBC_ENOMEM ? MFBC_OK : rc;
    }
    g->core = c;
    g->has_core = true;
    return MFBC_OK;
}

// Release a lane view: its workspace, counters and events (the device graph
// it shares stays with its owner).
void free_shadow(mfbc_graph *sh) {
    for (auto &e : sh->ev) {
        if (e) (void)hipEventDestroy(e);
        e = nullptr;
    }
    free_workspace(sh->ws);
    if (sh->h_ctr) (void)hipHostFree(sh->h_ctr);
    delete sh;
}

void free_graph_memory(mfbc_graph *g) {
    for (int i = 0; i < kMaxLanes; i++) {
        if (g->shadow[i]) free_shadow(g->shadow[i]);
        g->shadow[i] = nullptr;
        if (g->lane_stream[i]) (void)hipStreamDestroy(g->lane_stream[i]);
        g->lane_stream[i] = nullptr;
    }
    if (g->lane_start) (void)hipEventDestroy(g->lane_start);
    g->lane_start = nullptr;
    for (auto &e : g->ev) {
        if (e) (void)hipEventDestroy(e);
        e = nullptr;
    }
    g->timing = false;
    free_workspace(g->ws);
    if (g->has_core) free_view(g->core);
    g->core = View{};
    g->has_core = false;
    free_view(g->full);
    free_plans(g->own_out, g->own_in);
    dfree(g->perm);
    dfree(g->hub_dist);
    g->h_perm.clear();
    if (g->h_ctr) (void)hipHostFree(g->h_ctr);
    g->h_ctr = nullptr;
}

// Column groups of the workspace for MFBC over n_sources in batches of `batch`.
int bc_groups(int64_t n_sources, int32_t batch) {
    const int64_t width = std::max<int64_t>(1, std::min<int64_t>(batch, n_sources));
    return (int)((width + kWave - 1) / kWave);
}

// Algorithm 3 over the listed sources with the workspace already in place.
int bc_batches(mfbc_graph *g, const int32_t *d_sources, int64_t n_sources, int32_t batch, int ncg,
               double *d_bc, hipStream_t s) {
    g->stats = mfbc_stats{};
    launch_lambda_zero(g, ncg, s);
    int rc;
    for (int64_t b0 = 0; b0 < n_sources; b0 += batch) {
        const int nb = (int)std::min<int64_t>(batch, n_sources - b0);
        const int bcg = (nb + kWave - 1) / kWave;
        if ((rc = run_batch(g, bcg, nb, d_sources + b0, s))) return rc;
        g->stats.batches++;
    }
    launch_lambda_reduce(g, ncg, d_bc, s);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(s));
    return MFBC_OK;
}

// How the batches of one mfbc_bc call run when no lane count is set (a
// column depends on its own column of every product alone, Section 3), by the
// core's arcs times the column groups of one batch:
//  * up to 2^21, where a product is mostly latency: as one wide batch of four,
//    or of as many as keep the state within 256 MB, so a small graph's whole
//    source list shares each launch and read-back;
//  * up to 2^24: on four streams, each product large enough to fill the device
//    only partly;
//  * above: one after another, since the others gain little there for four
//    times the state.
// ms apart / on four streams / as one wide batch of four:
//   2^13    n = 1,024 of degree 8, 1,024 in batches of 64    9.6 / 2.9 / 2.8 (1.0 all in one)
//   2^19.2  weighted R-MAT scale 16, 1,024 in 256            6.2 / 3.6 / 3.9
//   2^20.8  unweighted R-MAT scale 16, 256 in 64             4.2 / 2.4 / 2.0
//   2^21.2  weighted R-MAT scale 18, 1,024 in 256           13.9 / 11.1 / 11.6
//   2^22.9  unweighted R-MAT scale 18, 256 in 64             8.6 / 7.7 / 5.9
//   2^23.3  weighted R-MAT scale 20, 1,024 in 256           37.0 / 32.4 / 33.2
//   2^23.8  unweighted R-MAT scale 16, 2,048 in 512         13.9 / 11.9 / 12.3
//   2^24.9  unweighted R-MAT scale 18, 1,024 in 256         21.8 / 21.3 / 20.6
// (batches of one group would rather be wide at 2^23, too; the rule does not
// look at the groups alone.)
// The state of batches that run together without being asked for stays within
// kLaneBytes (a sixth of a device's 288 GB; four lanes of 256 sources at n =
// 2^20 hold 42 GB): it is kept until the graph is freed.
constexpr double kLaneBytes = 48.0 * (1 << 30);

double column_bytes(const mfbc_graph *g) { return 39.0 * g->n + (double)g->core.arcs * 8.0 / kWave; }

// Batches of `ncg` groups whose state fits kLaneBytes, 1..kMaxLanes.
int lanes_within(const mfbc_graph *g, int ncg) {
    const double fit = kLaneBytes / (column_bytes(g) * kWave * ws_groups(ncg));
    return std::max(1, (int)std::min<double>(kMaxLanes, fit));
}

int64_t merged_batches(const mfbc_graph *g, int32_t batch, int ncg) {
    if ((double)g->core.arcs * (double)ncg > (double)(1 << 21)) return 1;
    const double fit = (double)(256 << 20) / column_bytes(g) / (double)batch;
    return std::max<int64_t>(lanes_within(g, ncg), (int64_t)fit);
}

// What products read of a graph, shared with g; the workspace, counters and
// statistics stay the view's own.
void share_graph(const mfbc_graph *g, mfbc_graph *to) {
    to->device = g->device;
    to->n = g->n;
    to->arcs = g->arcs;
    to->maxw = g->maxw;
    to->weighted = g->weighted;
    to->directed = g->directed;
    to->sparse = g->sparse;
    to->full = g->full;
    to->core = g->core;
    to->has_core = g->has_core;
    to->mb = g->mb;
    to->params = g->params;
    to->perm = g->perm;
}

// Lane i of g (i = 0: g itself), created on first use; a view is refreshed
// from g on every call (the plan may have changed).
int lane_graph(mfbc_graph *g, int i, mfbc_graph **out) {
    if (i == 0) {
        *out = g;
        return MFBC_OK;
    }
    mfbc_graph *&sh = g->shadow[i];
    if (!sh) {
        sh = new (std::nothrow) mfbc_graph();
        if (!sh) return fail(MFBC_ENOMEM, "host allocation failed");
        sh->is_shadow = true;
        if (hipHostMalloc((void **)&sh->h_ctr,
                          sizeof(unsigned long long) * kCounterWords) != hipSuccess) {
            sh->h_ctr = nullptr;
            delete sh;
            sh = nullptr;
            return fail(MFBC_ENOMEM, "pinned host allocation failed");
        }
    }
    if (!g->lane_stream[i]) HIP_TRY(hipStreamCreateWithFlags(&g->lane_stream[i], hipStreamNonBlocking));
    share_graph(g, sh);
    sh->timing = g->timing;
    if (g->timing && !sh->ev[0]) {
        for (auto &e : sh->ev) HIP_TRY(hipEventCreate(&e));
        for (int i = 0; i < 3 * kWindow; i++) sh->ev_pull[i] = i % 3 == 2 ? nullptr : sh->ev[i];
    }
    *out = sh;
    return MFBC_OK;
}

static_assert(sizeof(mfbc_stats) == 14 * sizeof(int64_t) + 9 * sizeof(double),
              "add_stats walks 14 counters and 9 times / byte counts");

void add_stats(mfbc_stats &a, const mfbc_stats &b) {
    int64_t *ai = &a.fwd_products;
    const int64_t *bi = &b.fwd_products;
    for (int k = 0; k < 14; k++) ai[k] += bi[k];
    double *ad = &a.fwd_pull_ms;
    const double *bd = &b.fwd_pull_ms;
    for (int k = 0; k < 9; k++) ad[k] += bd[k];
}

// lane(0) here and lane(1) .. lane(count - 1) on threads of their own; a lane
// whose thread cannot be started runs here after lane(0).
template <typename F>
void run_lanes(int count, const F &lane) {
    std::thread th[kMaxLanes];
    int started = 1;
    try {
        for (; started < count; started++) th[started] = std::thread(std::cref(lane), started);
    } catch (const std::exception &) {
    }
    lane(0);
    for (int i = started; i < count; i++) lane(i);
    for (auto &t : th)
        if (t.joinable()) t.join();
}

// Algorithm 3 with batch b on lane b % S: lane 0 on the caller's stream, the
// others on their own streams after the caller's prior work; each lane's
// host loop runs on its own thread; lambda = the lanes' parts, summed in lane
// order (so a call is deterministic for a given lane count).  `fewer`: lanes
// whose workspace does not fit are left out, down to the first.
int bc_lanes(mfbc_graph *g, const int32_t *d_sources, int64_t n_sources, int32_t batch, int ncg,
             int S, bool fewer, double *d_bc, hipStream_t s) {
    mfbc_graph *lg[kMaxLanes] = {};
    hipStream_t ls[kMaxLanes] = {};
    int rc;
    for (int i = 0; i < S; i++) {
        if ((rc = lane_graph(g, i, &lg[i]))) return rc;
        rc = ensure_workspace(lg[i], ncg);
        if (rc == MFBC_ENOMEM && fewer && i > 0) {
            S = i;
            break;
        }
        if (rc) return rc;
        ls[i] = i == 0 ? s : g->lane_stream[i];
    }
    if (!g->lane_start) HIP_TRY(hipEventCreateWithFlags(&g->lane_start, hipEventDisableTiming));
    HIP_TRY(hipEventRecord(g->lane_start, s));
    for (int i = 1; i < S; i++) HIP_TRY(hipStreamWaitEvent(ls[i], g->lane_start, 0));
    const int64_t nbat = (n_sources + batch - 1) / batch;
    int rcs[kMaxLanes] = {};
    std::string msgs[kMaxLanes];
    auto lane = [&](int i) {
        mfbc_graph *x = lg[i];
        int r = MFBC_OK;
        if (hipSetDevice(g->device) != hipSuccess) r = fail(MFBC_EDEVICE, "hipSetDevice failed");
        x->stats = mfbc_stats{};
        if (!r) launch_lambda_zero(x, ncg, ls[i]);
        for (int64_t b = i; !r && b < nbat; b += S) {
            const int64_t b0 = b * batch;
            const int nb = (int)std::min<int64_t>(batch, n_sources - b0);
            const int bcg = (nb + kWave - 1) / kWave;
            if (!r) r = run_batch(x, bcg, nb, d_sources + b0, ls[i]);
            x->stats.batches++;
        }
        if (!r && hipStreamSynchronize(ls[i]) != hipSuccess) r = fail(MFBC_EDEVICE, "lane stream failed");
        rcs[i] = r;
        if (r) msgs[i] = mfbc_last_error();
    };
    run_lanes(S, lane);
    for (int i = 0; i < S; i++)
        if (rcs[i]) return fail(rcs[i], msgs[i]);
    launch_lambda_reduce_lanes(lg, S, ncg, d_bc, s);
    mfbc_stats tot{};
    for (int i = 0; i < S; i++) add_stats(tot, lg[i]->stats);
    g->stats = tot;
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(s));
    return MFBC_OK;
}

// The workspace of `ncg` groups carved from `base` (same arrays and sizes as
// ensure_workspace allocates, each 256-byte aligned).
void carve_workspace(const mfbc_graph *g, int ncg, char *base, Workspace &ws) {
    ws = Workspace{};
    const int groups = ws_groups(ncg);
    size_t off = 0;
    ws.tau_words = (int)ws_tau_words(groups, false);
    ws_arrays(g, ws, groups, (size_t)ws.tau_words, [&](auto *&p, size_t count) {
        p = (std::remove_reference_t<decltype(p)>)(base + off);
        off = align256(off + std::max<size_t>(count, 1) * sizeof(*p));
    });
    ws.ncg = groups;
    ws.flags = (int32_t *)(ws.counters + kRingWords);
    ws.external = true;
}

// Swaps a graph's own workspace out for the duration of a call and back.
struct WorkspaceSwap {
    mfbc_graph *g;
    Workspace saved;
    explicit WorkspaceSwap(mfbc_graph *gr) : g(gr), saved(gr->ws) { g->ws = Workspace{}; }
    ~WorkspaceSwap() { g->ws = saved; }
};

// Whether the batched form's graphs run one after another on streams.  With T
// the sum over its two-group jobs of the graph's arcs and vertices and M the
// largest of them, the streams take about 230 us a graph and 2.2 ns an arc; the
// persistent launch the time of its largest job (eight waves: 1.5 us an
// of M) or, with every workgroup busy, 2.8 ns an arc.  Measured, streams /
// persistent, in ms:
//   3 graphs of 300                     0.9 / 2.0    32 of 200..6,000       27 / 98
//   8 of 200..1,000                     2.2 / 9.3    24 of 200..20,000     200 / 413
//   16 of 1,000..1,200, degree 40..64   4.9 / 19     64 of 200..20,000     330 / 498
//   40 of 200..2,000                     11 / 28     96 of 4,000..6,000    351 / 472
//   100 of 200..3,000                    38 / 58     200 of 200..1,000      46 / 23
//   64 of 1,000..1,200, degree 4..8      26 / 24.5   100 of 200..1,000      23 / 17
//   150 of 200..2,000                    42 / 42
bool many_underfilled(const std::vector<mfbc_graph *> &gs, const std::vector<int64_t> &ns) {
    double total = 0, most = 0;
    for (size_t i = 0; i < gs.size(); i++) {
        const double job = (double)gs[i]->core.arcs + gs[i]->n;
        total += job * (double)((ns[i] + 2 * kWave - 1) / (2 * kWave));
        if (ns[i]) most = std::max(most, job);
    }
    return 230e3 * (double)gs.size() + 2.2 * total < std::max(1500.0 * most, 2.8 * total);
}

// The batched form on streams: the graphs one after another on up to four,
// largest first, each with its sources in wide batches, so that a product
// spreads over the whole device instead of the eight waves of a job.  The
// state of the streams is carved from the batched form's scratch.  Each graph
// runs through a view of its handle, under the library's own decomposition of
// its core where mfbc_set_plan replaced that (run sizes tuned for the
// persistent launch's workgroups are too coarse for products that spread over
// the device: 32 graphs of 200..6,000 vertices took 50 ms under them, 29 under
// its own); the handle itself is only read, as by the persistent launch, so a
// server may step on it meanwhile.
constexpr size_t kManyLaneBytes = (size_t)512 << 20;

int many_on_streams(const std::vector<mfbc_graph *> &gs, const std::vector<const int32_t *> &src,
                    const std::vector<int64_t> &ns, const std::vector<double *> &out, size_t budget,
                    ManyWorkspace &mw, hipStream_t s, bool *done, unsigned long long *products) {
    *done = false;
    struct Item {
        mfbc_graph *g;
        mfbc_graph view;
        std::vector<size_t> at;      // positions in the call (a graph may be listed twice)
        int ncg;                     // column groups of a batch
        double cost;
    };
    std::vector<Item> items;
    for (size_t i = 0; i < gs.size(); i++) {
        Item *it = nullptr;
        for (auto &x : items)
            if (x.g == gs[i]) it = &x;
        if (!it) {
            items.push_back({gs[i], {}, {}, 1, 0.0});
            it = &items.back();
            share_graph(it->g, &it->view);
            it->view.h_ctr = it->g->h_ctr;
            if (it->g->own_out.tasks) {
                it->view.core.plan_out = it->g->own_out;
                it->view.core.plan_in = it->g->own_in;
            }
        }
        it->at.push_back(i);
        it->cost += (double)ns[i] * (double)(gs[i]->core.arcs + gs[i]->n);
    }
    size_t lane_bytes = 0;
    for (auto &x : items) {
        int64_t most = 0;
        for (size_t i : x.at) most = std::max(most, ns[i]);
        const int all = bc_groups(most, INT32_MAX);
        int batches = 1;
        x.ncg = all;
        while (x.ncg > 1 && ws_bytes(&x.view, x.ncg, false) > kManyLaneBytes) {
            batches++;
            x.ncg = (all + batches - 1) / batches;
        }
        lane_bytes = std::max(lane_bytes, ws_bytes(&x.view, x.ncg, false));
    }
    lane_bytes = align256(lane_bytes);
    const int lanes = (int)std::min<size_t>({(size_t)kMaxLanes, items.size(), budget / std::max<size_t>(lane_bytes, 1)});
    if (lanes < 1) return MFBC_OK;
    char *base = many_scratch(mw, lane_bytes * (size_t)lanes);
    if (!base) return MFBC_OK;
    std::stable_sort(items.begin(), items.end(), [](const Item &a, const Item &b) { return a.cost > b.cost; });
    mfbc_graph *g0 = gs[0];
    hipStream_t ls[kMaxLanes] = {s};
    if (!g0->lane_start) HIP_TRY(hipEventCreateWithFlags(&g0->lane_start, hipEventDisableTiming));
    HIP_TRY(hipEventRecord(g0->lane_start, s));
    for (int i = 1; i < lanes; i++) {
        if (!g0->lane_stream[i]) HIP_TRY(hipStreamCreateWithFlags(&g0->lane_stream[i], hipStreamNonBlocking));
        ls[i] = g0->lane_stream[i];
        HIP_TRY(hipStreamWaitEvent(ls[i], g0->lane_start, 0));
    }
    std::atomic<size_t> next{0};
    std::atomic<bool> stop{false};
    int rcs[kMaxLanes] = {};
    std::string msgs[kMaxLanes];
    std::atomic<unsigned long long> fwd{0}, bwd{0};
    auto lane = [&](int i) {
        int rc = hipSetDevice(g0->device) == hipSuccess ? MFBC_OK : fail(MFBC_EDEVICE, "hipSetDevice failed");
        while (!rc && !stop) {
            const size_t k = next++;
            if (k >= items.size()) break;
            Item &x = items[k];
            carve_workspace(&x.view, x.ncg, base + (size_t)i * lane_bytes, x.view.ws);
            for (size_t at : x.at) {
                if (rc) break;
                rc = bc_batches(&x.view, src[at], ns[at], x.ncg * kWave, bc_groups(ns[at], x.ncg * kWave), out[at],
                                ls[i]);
                fwd += (unsigned long long)x.view.stats.fwd_products;
                bwd += (unsigned long long)x.view.stats.bwd_products;
            }
        }
        if (rc) {
            stop = true;
            msgs[i] = mfbc_last_error();
            (void)hipStreamSynchronize(ls[i]);
        }
        rcs[i] = rc;
    };
    run_lanes(lanes, lane);
    for (int i = 0; i < lanes; i++)
        if (rcs[i]) return fail(rcs[i], msgs[i]);
    products[0] += fwd;
    products[1] += bwd;
    *done = true;
    return MFBC_OK;
}

// Address of the static scratch on `device` (which must be current): taken
// once per device with hipGetSymbolAddress and kept.  Host code never uses
// the array's own name as an address.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char *g_scratch_base[kMaxDevices] = {};

int scratch_base(int device, char **out) {
    if (device < 0 || device >= kMaxDevices) return fail(MFBC_EDEVICE, "device index out of range");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_base[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(MFBC_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch_base[device] = (char *)p;
    }
    *out = g_scratch_base[device];
    return MFBC_OK;
}

}  // namespace

extern "C" {

const char *mfbc_last_error(void) { return g_err.c_str(); }

int mfbc_load_graph(int32_t n, int64_t n_arcs, const int64_t *h_row_ptr, const int32_t *h_col_idx,
                    const int32_t *h_weight, uint32_t flags, void *hip_stream, mfbc_graph **out) {
    if (!out) return fail(MFBC_EINVAL, "out is NULL");
    *out = nullptr;
    const uint32_t kind = flags & ~(uint32_t)MFBC_KEEP_ORDER;
    if (kind != MFBC_UNDIRECTED && kind != MFBC_DIRECTED)
        return fail(MFBC_EINVAL, "flags must be MFBC_UNDIRECTED or MFBC_DIRECTED "
                                 "(optionally | MFBC_KEEP_ORDER)");
    int32_t maxw = 1;
    {
        std::string msg;
        const int vrc = validate_csr(n, n_arcs, h_row_ptr, h_col_idx, h_weight, &maxw, msg);
        if (vrc) return fail(vrc, msg);
    }
    std::vector<int64_t> rpt;
    std::vector<int32_t> colt, wt;
    build_transpose(n, n_arcs, h_row_ptr, h_col_idx, h_weight, rpt, colt, wt);
    const bool directed = kind == MFBC_DIRECTED;
    if (!directed && !is_symmetric(n, n_arcs, h_row_ptr, h_col_idx, h_weight, rpt, colt, wt))
        return fail(MFBC_EINVAL, "undirected graph must have a symmetric CSR with equal weights");
    // device numbering: out-arcs (rp_o, col_o, w_o) and in-arcs (rpt, colt, wt)
    const int64_t *rp_o = h_row_ptr;
    const int32_t *col_o = h_col_idx, *w_o = h_weight;
    std::vector<int32_t> perm, iperm;
    std::vector<int64_t> rpo;
    std::vector<int32_t> colo, wo;
    if (!(flags & MFBC_KEEP_ORDER)) {
        degree_order(n, n_arcs, h_row_ptr, h_col_idx, perm, iperm);
        relabel_reverse(n, n_arcs, h_row_ptr, h_col_idx, h_weight, perm, iperm, rpt, colt, wt);
        if (directed) {
            build_transpose(n, n_arcs, rpt.data(), colt.data(), h_weight ? wt.data() : nullptr,
                            rpo, colo, wo);
            rp_o = rpo.data();
            col_o = colo.data();
            w_o = h_weight ? wo.data() : nullptr;
        } else {
            rp_o = rpt.data();
            col_o = colt.data();
            w_o = h_weight ? wt.data() : nullptr;
        }
    }
    mfbc_graph *g = new (std::nothrow) mfbc_graph();
    if (!g) return fail(MFBC_ENOMEM, "host allocation failed");
    if (hipGetDevice(&g->device) != hipSuccess) {
        delete g;
        return fail(MFBC_EDEVICE, "no HIP device");
    }
    g->n = n;
    g->arcs = n_arcs;
    g->maxw = maxw;
    g->weighted = h_weight != nullptr;
    g->directed = directed;
    // packed frontier tuples: weight bits for (n - 1) * max weight (+1 so that
    // no tuple equals the all-ones "absent" marker), the rest for multiplicities
    g->mb = 32 - bits_for((int64_t)(n - 1) * maxw + 1);
    int rc = upload_csr(n, n_arcs, rp_o, col_o, w_o, maxw, g->full.out);
    if (!rc) {
        if (directed)
            rc = upload_csr(n, n_arcs, rpt.data(), colt.data(), h_weight ? wt.data() : nullptr,
                            maxw, g->full.in);
        else
            g->full.in = g->full.out;
    }
    if (!rc && !perm.empty()) {
        if (!(rc = dalloc(&g->perm, (size_t)n))) {
            if (hipMemcpy(g->perm, perm.data(), (size_t)n * sizeof(int32_t),
                          hipMemcpyHostToDevice) != hipSuccess)
                rc = fail(MFBC_EDEVICE, "copy of the vertex order failed");
            g->h_perm = std::move(perm);
        }
    }
    g->h_rp_out.assign(rp_o, rp_o + (size_t)n + 1);
    g->h_rp_in = directed ? rpt : g->h_rp_out;
    if (!rc && hipHostMalloc((void **)&g->h_ctr,
                             sizeof(unsigned long long) * kCounterWords) != hipSuccess) {
        g->h_ctr = nullptr;
        rc = fail(MFBC_ENOMEM, "pinned host allocation failed");
    }
    g->full.arcs = n_arcs;
    if (!rc) rc = plan_views(g, TaskParams{0, 0, 0, 0});
    if (!rc) g->sparse = sparse_rows(g);
    if (!rc && core_worth_trying(g)) rc = build_core(g, (hipStream_t)hip_stream);
    if (rc) {
        free_graph_memory(g);
        delete g;
        return rc;
    }
    *out = g;
    return MFBC_OK;
}

int mfbc_free_graph(mfbc_graph *g) {
    if (!g) return MFBC_OK;
    // a live server holds the graph's CSR, plan and its own back pointer
    if (g->servers > 0)
        return fail(MFBC_EINVAL, "the graph has live servers (mfbc_server_create); free them "
                                 "before the graph");
    DeviceGuard dg(g->device);
    (void)hipDeviceSynchronize();
    free_graph_memory(g);
    delete g;
    return MFBC_OK;
}

int mfbc_forward(mfbc_graph *g, const int32_t *d_sources, int32_t nb, int32_t *d_dist,
                 double *d_sigma, int32_t *h_products, void *hip_stream) {
    return forward_impl(g, d_sources, nb, d_dist, d_sigma, false, nullptr, nullptr, nullptr, 0,
                        h_products, hip_stream);
}

int mfbc_fixpoint(mfbc_graph *g, int32_t op, const int32_t *d_sources, int32_t nb,
                  void *d_out, int32_t *h_products, void *hip_stream) {
    if (!g) return fail(MFBC_EINVAL, "graph handle is NULL");
    if (!mono_op_known(op)) return fail(MFBC_EINVAL, "unknown operation");
    if (nb < 1) return fail(MFBC_EINVAL, "nb must be >= 1");
    if (!d_out) return fail(MFBC_EINVAL, "output pointer is NULL");
    if (!d_sources) return fail(MFBC_EINVAL, "sources pointer is NULL");
    DeviceGuard dg(g->device);
    hipStream_t s = (hipStream_t)hip_stream;
    int rc;
    const int ncg = (nb + kWave - 1) / kWave;
    if ((rc = ensure_workspace(g, ncg))) return rc;
    g->stats = mfbc_stats{};
    const bool bits = bits_fit(g, op);
    Begun begun;
    if (op == MFBC_OP_SSSP && !bits) {
        bool fits = false;
        int32_t products = 0;
        if ((rc = run_quad(g, false, false, ncg, nb, d_sources, &products, &fits, &begun, s))) return rc;
        if (fits) {
            g->stats.batches = 1;
            if (h_products) *h_products = products;
            launch_quad_rows(g, false, ncg, nb, (int32_t *)d_out, nullptr, s);
            HIP_TRY(hipGetLastError());
            HIP_TRY(hipStreamSynchronize(s));
            return MFBC_OK;
        }
    }
    if (bits) launch_bits_init(g, ncg, nb, d_sources, s);
    else if (!begun.j) launch_mono_init(g, op, ncg, nb, d_sources, s);
    int planes = 0;              // planes of the product number cleared so far
    const double arc_bytes = g->weighted && op != MFBC_OP_BFS ? 8.0 : 4.0;
    mfbc_stats &st = g->stats;
    int64_t prev = begun.j ? begun.prev : nb;
    int j = begun.j, last = 0;
    // windows of products with one counter read-back each, as in MFBF
    while (!last) {
        if (j > g->n + 1) return fail(MFBC_EDEVICE, "fixpoint products did not converge");
        if (bits) {
            const int need = bits_for(j + kWindow);
            launch_bits_planes(g, ncg, planes, need, s);
            planes = need;
        }
        for (int i = 0; i < kWindow; i++) {
            if (bits) launch_bits_product(g, ncg, j + 1 + i, s, window_events(g, i, true));
            else launch_mono_product(g, op, ncg, j + 1 + i, s, window_events(g, i, true));
        }
        if ((rc = read_ring(g, s))) return rc;
        if (j == 0 && ring_flag(g, 2)) return bad_source(g, d_sources, nb, s);
        for (int i = 0; i < kWindow; i++) {
            const int jj = j + 1 + i;
            st.fwd_pull_launches++;
            add_times(g, i, &st.fwd_pull_ms, &st.fwd_merge_ms, true);
            if (last) continue;
            const Counts c = ring_counts(g, jj);
            st.fwd_entries += c.produced;
            st.fwd_outputs += c.outputs;
            st.fwd_active_vertices += c.active_vertices;
            st.fwd_active_arcs += c.active_arcs;
            // adjacency of the active rows, frontier values read once, T read
            // where a candidate arrived, T and the next frontier written per entry
            st.fwd_alg_bytes += 8.0 * c.active_vertices + arc_bytes * c.active_arcs +
                                4.0 * (double)(prev + c.outputs) + 8.0 * (double)c.produced;
            prev = c.produced;
            if (c.produced == 0) last = jj;
        }
        j += kWindow;
    }
    j = last;
    st.fwd_products = j;
    st.batches = 1;
    if (h_products) *h_products = j;
    // 4-byte values whatever their type: the tile export copies them as int32
    if (bits) launch_bits_export(g, op, ncg, nb, bits_for(last), d_out, s);
    else launch_export_tiles_i32(g, ncg, nb, g->ws.tdist, (int32_t *)d_out, s);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(s));
    return MFBC_OK;
}

int mfbc_forward_trace(mfbc_graph *g, const int32_t *d_sources, int32_t nb, int32_t *d_dist,
                       double *d_sigma, uint64_t *d_fbits, int32_t max_products, int64_t *h_nnz,
                       int64_t *h_relax, int32_t *h_products, void *hip_stream) {
    return forward_impl(g, d_sources, nb, d_dist, d_sigma, true, d_fbits, h_nnz, h_relax,
                        max_products, h_products, hip_stream);
}

int mfbc_backward(mfbc_graph *g, const int32_t *d_sources, int32_t nb, const int32_t *d_dist,
                  const double *d_sigma, double *d_delta, int32_t *h_products, void *hip_stream) {
    return backward_impl(g, d_sources, nb, d_dist, d_sigma, d_delta, nullptr, h_products,
                         hip_stream);
}

int mfbc_backward_trace(mfbc_graph *g, const int32_t *d_sources, int32_t nb, const int32_t *d_dist,
                        const double *d_sigma, double *d_delta, int32_t *d_step,
                        int32_t *h_products, void *hip_stream) {
    if (!d_step) return fail(MFBC_EINVAL, "d_step is NULL");
    return backward_impl(g, d_sources, nb, d_dist, d_sigma, d_delta, d_step, h_products,
                         hip_stream);
}

int mfbc_bc(mfbc_graph *g, const int32_t *d_sources, int64_t n_sources, int32_t batch,
            double *d_bc, void *hip_stream) {
    if (!g) return fail(MFBC_EINVAL, "graph handle is NULL");
    if (n_sources < 0) return fail(MFBC_EINVAL, "n_sources must be >= 0");
    if (batch < 1) return fail(MFBC_EINVAL, "batch must be >= 1");
    if (!d_bc) return fail(MFBC_EINVAL, "d_bc is NULL");
    DeviceGuard dg(g->device);
    hipStream_t s = (hipStream_t)hip_stream;
    if (n_sources > 0 && !d_sources) return fail(MFBC_EINVAL, "sources pointer is NULL");
    int rc;
    const int ncg = bc_groups(n_sources, batch);
    const int64_t nbat = (n_sources + batch - 1) / batch;
    const double work = (double)g->core.arcs * (double)ncg;
    const int lanes =
        g->lanes ? g->lanes : (work > (double)(1 << 21) && work <= (double)(1 << 24) ? lanes_within(g, ncg) : 1);
    if (lanes > 1 && nbat > 1) {
        if ((rc = check_sources(g, d_sources, n_sources, s))) return rc;
        return bc_lanes(g, d_sources, n_sources, batch, ncg, (int)std::min<int64_t>(lanes, nbat), g->lanes == 0, d_bc,
                        s);
    }
    const int64_t wide = g->lanes ? 1 : std::min(nbat, merged_batches(g, batch, ncg));
    if (wide > 1) {
        const int64_t cols = std::min<int64_t>(n_sources, wide * batch);
        const int wcg = bc_groups(n_sources, (int32_t)cols);
        rc = ensure_workspace(g, wcg);
        if (!rc) {
            rc = bc_batches(g, d_sources, n_sources, (int32_t)cols, wcg, d_bc, s);
            g->stats.batches = nbat;
            return rc;
        }
        if (rc != MFBC_ENOMEM) return rc;      // else as the caller sized it
    }
    if ((rc = ensure_workspace(g, ncg))) return rc;
    return bc_batches(g, d_sources, n_sources, batch, ncg, d_bc, s);
}

int mfbc_bc_requests(mfbc_graph *g, const int32_t *d_sources, const int64_t *h_first,
                     int32_t n_requests, int32_t batch, double *const *h_out, void *hip_stream) {
    if (!g) return fail(MFBC_EINVAL, "graph handle is NULL");
    if (n_requests < 0) return fail(MFBC_EINVAL, "n_requests must be >= 0");
    if (batch < kWave || batch % kWave || batch > kWave * kMaxBatchGroups)
        return fail(MFBC_EINVAL, "batch must be a multiple of 64 in [64, 4096]");
    if (n_requests == 0) return MFBC_OK;
    if (!h_first || !h_out) return fail(MFBC_EINVAL, "h_first or h_out is NULL");
    if (h_first[0] != 0) return fail(MFBC_EINVAL, "h_first[0] must be 0");
    for (int32_t r = 0; r < n_requests; r++) {
        if (h_first[r + 1] < h_first[r]) return fail(MFBC_EINVAL, "h_first must be non-decreasing");
        if (!h_out[r]) return fail(MFBC_EINVAL, "an output pointer is NULL");
    }
    const int64_t total = h_first[n_requests];
    if (total > 0 && !d_sources) return fail(MFBC_EINVAL, "d_sources is NULL");
    DeviceGuard dg(g->device);
    hipStream_t s = (hipStream_t)hip_stream;
    int rc = check_sources(g, d_sources, total, s);
    if (rc) return rc;
    // every request's sources in whole column groups, requests in list order
    struct Slot {
        int64_t first;
        int32_t count, req;
    };
    std::vector<Slot> slots;
    for (int32_t r = 0; r < n_requests; r++)
        for (int64_t k = h_first[r]; k < h_first[r + 1]; k += kWave)
            slots.push_back({k, (int32_t)std::min<int64_t>(kWave, h_first[r + 1] - k), r});
    for (int32_t r = 0; r < n_requests; r++) launch_zero_f64(h_out[r], (size_t)g->n, s);
    const int G = batch / kWave;
    const int ncg = (int)std::min<size_t>((size_t)G, slots.size());
    g->stats = mfbc_stats{};
    if (ncg > 0 && (rc = ensure_workspace(g, ncg))) return rc;
    for (size_t b0 = 0; b0 < slots.size(); b0 += (size_t)G) {
        const int bcg = (int)std::min<size_t>((size_t)G, slots.size() - b0);
        GroupSpans sp{};
        GroupOuts o{};
        for (int cg = 0; cg < bcg; cg++) {
            sp.first[cg] = slots[b0 + cg].first;
            sp.count[cg] = slots[b0 + cg].count;
            o.out[cg] = h_out[slots[b0 + cg].req];
        }
        launch_set_sources_spans(g, bcg, d_sources, sp, s);
        launch_lambda_zero(g, bcg, s);
        // padding columns (source -1) seed nothing and reach nothing
        if ((rc = run_batch(g, bcg, bcg * kWave, nullptr, s))) return rc;
        launch_lambda_add_groups(g, bcg, o, s);
        g->stats.batches++;
    }
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(s));
    return MFBC_OK;
}

int mfbc_set_lanes(mfbc_graph *g, int32_t lanes) {
    if (!g) return fail(MFBC_EINVAL, "graph handle is NULL");
    if (lanes < 0 || lanes > kMaxLanes)
        return fail(MFBC_EINVAL, "lanes must be in [0, " + std::to_string(kMaxLanes) + "]");
    g->lanes = lanes;
    return MFBC_OK;
}

int mfbc_bc_noalloc(mfbc_graph *g, const int32_t *d_sources, int64_t n_sources, int32_t batch,
                    double *d_bc, void *hip_stream) {
    if (!g) return fail(MFBC_EINVAL, "graph handle is NULL");
    if (n_sources < 0) return fail(MFBC_EINVAL, "n_sources must be >= 0");
    if (batch < 1) return fail(MFBC_EINVAL, "batch must be >= 1");
    if (!d_bc) return fail(MFBC_EINVAL, "d_bc is NULL");
    if (n_sources > 0 && !d_sources) return fail(MFBC_EINVAL, "sources pointer is NULL");
    DeviceGuard dg(g->device);
    hipStream_t s = (hipStream_t)hip_stream;
    int ncg = bc_groups(n_sources, batch);
    const int64_t nbat = (n_sources + batch - 1) / batch;
    const size_t need = ws_bytes(g, ncg, true);
    if (need > kScratchBytes)
        return fail(MFBC_ENOMEM, "mfbc_bc_noalloc: this graph and batch need " + std::to_string(need) +
                                     " bytes of workspace; the static scratch holds " +
                                     std::to_string(kScratchBytes));
    // where the finer row cut's partials do not fit beside the batch, it runs in
    // parts (lambda is a sum over sources)
    while (ncg > 1 && ws_bytes(g, ncg, false) > kScratchSize) {
        ncg /= 2;
        batch = ncg * kWave;
    }
    // several batches as one wide one while they fit, as in mfbc_bc
    while (!g->lanes && ncg * (int64_t)kWave < n_sources && ws_bytes(g, 2 * ncg, false) <= kScratchSize) {
        ncg = (int)std::min<int64_t>(2 * ncg, bc_groups(n_sources, INT32_MAX));
        batch = ncg * kWave;
    }
    if (ws_bytes(g, ncg, false) > kScratchSize)
        return fail(MFBC_ENOMEM, "mfbc_bc_noalloc: the hub partials of this graph's plan do not fit the scratch");
    char *base = nullptr;
    int rc = scratch_base(g->device, &base);
    if (rc) return rc;
    // the caller's workspace stays untouched: the batch state is carved from
    // the scratch and swapped in for the duration of the call
    WorkspaceSwap sw(g);
    carve_workspace(g, ncg, base, g->ws);
    // sources are checked on the device (no host copy of the list)
    launch_check_sources(d_sources, n_sources, g->n, g->ws.flags + 1, s);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpyAsync(g->h_ctr, g->ws.flags + 1, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (*(const int32_t *)g->h_ctr != 0) return fail(MFBC_EINVAL, "a source is outside [0, n)");
    rc = bc_batches(g, d_sources, n_sources, batch, ncg, d_bc, s);
    g->stats.batches = nbat;
    return rc;
}

int mfbc_set_plan(mfbc_graph *g, int32_t run_arcs, int32_t run_verts, int32_t heavy,
                  int32_t slice) {
    if (!g) return fail(MFBC_EINVAL, "graph handle is NULL");
    if (run_verts > 64) return fail(MFBC_EINVAL, "run_verts must be <= 64");
    // a run's arcs are addressed with 32-bit offsets in the kernels
    if (run_arcs > (1 << 24) || heavy > (1 << 24) || slice > (1 << 24))
        return fail(MFBC_EINVAL, "run_arcs, heavy and slice must be <= 2^24");
    // a server sizes its hub partials by the plan it was created with
    if (g->servers > 0)
        return fail(MFBC_EINVAL, "the graph has live servers (mfbc_server_create); free them "
                                 "before changing its plan");
    DeviceGuard dg(g->device);
    HIP_TRY(hipDeviceSynchronize());
    const int32_t old_slots = max_slots(g);
    const int rc = plan_views(g, TaskParams{run_arcs, run_verts, heavy, slice});
    if (rc) return rc;
    // the partial buffers are sized by the slot count: regrow on next use
    if (max_slots(g) > old_slots) {
        free_workspace(g->ws);
        for (auto *sh : g->shadow)
            if (sh) free_workspace(sh->ws);
    }
    return MFBC_OK;
}

int mfbc_enable_timing(mfbc_graph *g, int enable) {
    if (!g) return fail(MFBC_EINVAL, "graph handle is NULL");
    if (enable < 0 || enable > 2) return fail(MFBC_EINVAL, "enable must be 0, 1 or 2");
    DeviceGuard dg(g->device);
    if (enable && !g->ev[0]) {
        for (auto &e : g->ev) HIP_TRY(hipEventCreate(&e));
        for (int i = 0; i < 3 * kWindow; i++) g->ev_pull[i] = i % 3 == 2 ? nullptr : g->ev[i];
    }
    g->timing = g->ev[0] != nullptr ? enable : 0;
    return MFBC_OK;
}

int mfbc_bc_many(int32_t n_graphs, mfbc_graph *const *graphs, const int32_t *const *d_sources,
                 const int64_t *h_n_sources, double *const *d_bc, const mfbc_many_config *config,
                 mfbc_stats *h_stats, void *hip_stream) {
    if (n_graphs < 0) return fail(MFBC_EINVAL, "n_graphs must be >= 0");
    if (n_graphs == 0) return MFBC_OK;
    if (!graphs || !d_sources || !h_n_sources || !d_bc)
        return fail(MFBC_EINVAL, "array argument is NULL");
    const int dev = graphs[0] ? graphs[0]->device : 0;
    std::vector<mfbc_graph *> gs((size_t)n_graphs);
    std::vector<const int32_t *> src((size_t)n_graphs);
    std::vector<int64_t> ns((size_t)n_graphs);
    std::vector<double *> out((size_t)n_graphs);
    for (int32_t i = 0; i < n_graphs; i++) {
        if (!graphs[i]) return fail(MFBC_EINVAL, "graph " + std::to_string(i) + " is NULL");
        if (graphs[i]->device != dev) return fail(MFBC_EINVAL, "graphs live on different devices");
        if (h_n_sources[i] < 0) return fail(MFBC_EINVAL, "negative source count");
        if (!d_bc[i]) return fail(MFBC_EINVAL, "output " + std::to_string(i) + " is NULL");
        gs[(size_t)i] = graphs[i];
        src[(size_t)i] = d_sources[i];
        ns[(size_t)i] = h_n_sources[i];
        out[(size_t)i] = d_bc[i];
    }
    int block_threads = config && config->block_threads ? config->block_threads : 512;
    if (block_threads != 256 && block_threads != 512)
        return fail(MFBC_EINVAL, "block_threads must be 256 or 512");
    const int job_width = config && config->job_width ? config->job_width : kWave;
    if (job_width != kWave && job_width != 2 * kWave)
        return fail(MFBC_EINVAL, "job_width must be 64 or 128");
    const int w = job_width / kWave;
    DeviceGuard dg(dev);
    hipStream_t s = (hipStream_t)hip_stream;
    int rc;
    for (int32_t i = 0; i < n_graphs; i++)
        if ((rc = check_sources(gs[(size_t)i], src[(size_t)i], ns[(size_t)i], s))) return rc;
    int cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    const int full = (2048 / block_threads) * cus;       // 8 waves per SIMD
    int blocks = config && config->blocks > 0 ? config->blocks : full;
    // fewer workgroups than fill the device: the caller leaves the rest of it to
    // others, which the streams would take
    const bool shared = blocks < full;
    int n_max = 1, slots_max = 1;
    int64_t arcs_max = 1;
    for (auto *g : gs) {
        n_max = std::max(n_max, g->n);
        slots_max = std::max(slots_max, max_slots(g));
        arcs_max = std::max<int64_t>(arcs_max, g->core.arcs);
    }
    size_t free_b = 0, total_b = 0;
    HIP_TRY(hipMemGetInfo(&free_b, &total_b));
    const size_t slot = many_slot_bytes(n_max, slots_max, arcs_max, w);
    ManyWorkspace &ws = many_workspace(dev);
    // half of the memory free or already held by the workspace: the same cap
    // on every call, so a first call runs with the block count of later ones
    const size_t budget = (free_b + ws_scratch_bytes(ws)) / 2;
    const int cap = (int)std::max<size_t>(1, budget / std::max<size_t>(slot, 1));
    blocks = std::min(blocks, cap);
    unsigned long long tot[2] = {0, 0};
    bool done = false;
    if (!shared && many_underfilled(gs, ns) && (rc = many_on_streams(gs, src, ns, out, budget, ws, s, &done, tot))) return rc;
    // one persistent launch per arc encoding (unweighted, packed, separate)
    for (int mode = 0; mode < 3 && !done; mode++) {
        std::vector<mfbc_graph *> g2;
        std::vector<const int32_t *> s2;
        std::vector<int64_t> n2;
        std::vector<double *> o2;
        for (size_t i = 0; i < gs.size(); i++) {
            const Csr &c = gs[i]->core.in;
            const int m = c.pk ? 1 : (c.w ? 2 : 0);
            if (m != mode) continue;
            g2.push_back(gs[i]);
            s2.push_back(src[i]);
            n2.push_back(ns[i]);
            o2.push_back(out[i]);
        }
        if (g2.empty()) continue;
        unsigned long long st[2] = {0, 0};
        int32_t flags[2] = {0, 0};
        std::string err;
        rc = launch_bc_many(g2, s2, n2, o2, block_threads, blocks, w, s, ws, st, flags, err);
        if (rc) return fail(rc, err);
        if (flags[1]) return fail(MFBC_EDEVICE, "products did not converge");
        if (flags[0]) return fail(MFBC_EOVERFLOW, "a shortest-path count overflowed binary64");
        tot[0] += st[0];
        tot[1] += st[1];
    }
    if (h_stats) {
        *h_stats = mfbc_stats{};
        h_stats->fwd_products = (int64_t)tot[0];
        h_stats->bwd_products = (int64_t)tot[1];
    }
    return MFBC_OK;
}

int mfbc_get_stats(const mfbc_graph *g, mfbc_stats *out) {
    if (!g || !out) return fail(MFBC_EINVAL, "NULL argument");
    *out = g->stats;
    return MFBC_OK;
}

int mfbc_graph_info(const mfbc_graph *g, int32_t *n, int64_t *n_arcs, int32_t *max_weight) {
    if (!g) return fail(MFBC_EINVAL, "graph handle is NULL");
    if (n) *n = g->n;
    if (n_arcs) *n_arcs = g->arcs;
    if (max_weight) *max_weight = g->maxw;
    return MFBC_OK;
}

}  // extern "C"
