// The shortest-path core of a weighted graph: the arcs that can lie on a
// shortest path.  An arc u -> v of weight w is on none if some walk from u to
// v is lighter, and a walk through a landmark l shows that without a search:
// with upper bounds to[u][l] >= d(u, l) and from[v][l] >= d(l, v), the arc goes
// if to[u][l] + from[v][l] < w for any l (the walk cannot use the arc itself,
// it would weigh w or more).  What is kept therefore holds every shortest path
// of the graph, so distances, path counts, the shortest-path DAG and the
// dependencies computed over it are those of the whole graph.
//
// With integer weights drawn from a wide range most arcs go: 64 landmarks
// leave 8% of the arcs of a weighted R-MAT graph (edge factor 16, weights
// 1..255) and 7% of a uniform graph of degree 256, and every product, the
// counting product and the stored DAG shrink with them.
//
// The landmarks are the vertices of highest degree, one per lane, and the
// bounds one 64-column run of the fixpoint product (min, a + w) stopped after
// six products: an unfinished run leaves weights of walks, which
// are upper bounds all the same.
#include <algorithm>

#include "pull.h"

namespace mfbc {
namespace {

constexpr uint32_t kFar = (uint32_t)kInf;

// One wave per task of the decomposition: lane l holds landmark l's bound of
// the row's vertex and gathers the other end's row of bounds (256 B) for every
// arc, eight in flight; the arc is dropped if any lane finds a lighter walk.
// Bound by the gathers: one per arc, of rows that the degree order packs.
template <int AM>
__global__ __launch_bounds__(kBlock) void k_core_mark(const Task *tasks, int ntasks, const int64_t *rp,
                                                      ArcSrc arcs, const uint32_t *near,
                                                      const uint32_t *far, uint8_t *keep, int32_t *cnt) {
    constexpr int U = 8;
    const int lane = threadIdx.x & (kWave - 1);
    const int t = blockIdx.x * kWavesPerBlock + uni((int)(threadIdx.x >> 6));
    if (t >= ntasks) return;
    const Task *tp = tasks + t;
    const int v0 = uni(tp->v0), v1 = uni(tp->v1), hub = uni(tp->hub);
    const int64_t e0 = uni64(tp->e0), e1 = uni64(tp->e1);
    for (int x = v0; x < v1; x++) {
        const uint32_t dx = near[(size_t)x * kWave + lane];
        const int64_t ea = hub >= 0 ? e0 : rp[x], eb = hub >= 0 ? e1 : rp[x + 1];
        int kept = 0;
        for (int64_t e = ea; e < eb; e += kWave) {
            const int64_t my = e + lane;
            int y = 0, w = 0;
            if (my < eb) load_arc<AM>(arcs, my, y, w);
            const int n = (int)(eb - e < kWave ? eb - e : kWave);
            uint64_t on = 0;
            for (int j = 0; j < n; j += U) {
                uint32_t d[U];
#pragma unroll
                for (int k = 0; k < U; k++) {
                    d[k] = kFar;
                    if (j + k < n) d[k] = far[(size_t)(uint32_t)rdlane(y, j + k) * kWave + lane];
                }
#pragma unroll
                for (int k = 0; k < U; k++)
                    if (j + k < n) {
                        // unreached bounds are 2^31 - 1: the sum of two fits 32 bits
                        const bool lighter = dx + d[k] < (uint32_t)rdlane(w, j + k);
                        if (!ballot(lighter)) on |= 1ull << (j + k);
                    }
            }
            if (my < eb) keep[my] = (uint8_t)((on >> lane) & 1ull);
            kept += __popcll(on);
        }
        if (lane == 0) {
            if (hub >= 0) atomicAdd(cnt + x, kept);      // a slice: the row's count is the slices' sum
            else cnt[x] = kept;
        }
    }
}

__global__ void k_core_zero(int32_t *cnt, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) cnt[i] = 0;
}

__global__ void k_core_hub(const int32_t *bound, int n, int32_t *out) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n) out[v] = bound[(size_t)v * kWave];
}

// One wave per row: the kept arcs in their order, to the row's place in `out`.
__global__ __launch_bounds__(kBlock) void k_core_compact(int n, Csr c, const uint8_t *keep, Csr out) {
    const int lane = threadIdx.x & (kWave - 1);
    const int x = blockIdx.x * kWavesPerBlock + uni((int)(threadIdx.x >> 6));
    if (x >= n) return;
    int64_t to = out.rp[x];
    const int64_t eb = c.rp[x + 1];
    for (int64_t e = c.rp[x]; e < eb; e += kWave) {
        const int64_t my = e + lane;
        const bool on = my < eb && keep[my] != 0;
        const uint64_t m = ballot(on);
        if (on) {
            const int64_t p = to + __popcll(m & ((1ull << lane) - 1ull));
            if (c.pk) {
                out.pk[p] = c.pk[my];
            } else {
                out.col[p] = c.col[my];
                out.w[p] = c.w[my];
            }
        }
        to += __popcll(m);
    }
}

}  // namespace

// Whether the run over the landmarks can pay: some weight above 1, more than a
// few arcs, and many ways around an arc, by the mean degree of an arc's end
// (sum of squared degrees over their sum).  Kept share of the arcs measured
// on weights 1..100 / 1..255: uniform graphs of degree 12 (mean 13) 85%, 20
// 56%, 40 31%; R-MAT graphs of edge factor 2 (mean 70) 34%, 4 22%, 16 8%.
bool core_worth_trying(const mfbc_graph *g) {
    return g->weighted && g->maxw > 1 && g->arcs >= 2048 && !g->sparse;
}

bool sparse_rows(const mfbc_graph *g) {
    double sq = 0.0;
    for (int32_t v = 0; v < g->n; v++) {
        const double d = (double)(g->h_rp_out[(size_t)v + 1] - g->h_rp_out[(size_t)v]);
        sq += d * d;
    }
    return sq < 16.0 * (double)g->arcs;
}

// A core's rows are short (2.5 arcs on average at R-MAT scale 20), so a run
// holds at least 16 rows for its fixed cost, and its longest rows, one wave
// each, would be the tail of every product: they are cut from 256 arcs on.
// Measured, ms per pass, four rows a run and rows cut from 1024 arcs on /
// these: directed R-MAT n = 100,003, 300 sources 3.84 / 2.92; dependencies of
// 130 sources at R-MAT scale 18 2.43 / 2.26; 256 sources at scale 20 the same
// 16.5, where a run has 64 rows either way.
TaskParams core_params(int32_t n, int64_t arcs, int64_t full_arcs) {
    constexpr int64_t kTarget = 16384;
    TaskParams p;
    p.run_verts = (int)std::min<int64_t>(64, std::max<int64_t>(16, (n + kTarget - 1) / kTarget));
    p.run_arcs = (int)std::min<int64_t>(256, std::max<int64_t>(64, (arcs + kTarget - 1) / kTarget));
    // (longer slices for a core of most arcs: its DAG masks and partials stay
    // within the memory of the whole graph's masks)
    p.slice = 15 * full_arcs < 32 * arcs ? 256 : 128;
    p.heavy = 2 * p.slice;
    return p;
}

void launch_core_mark(const Csr &c, const Plan &pl, const int32_t *near, const int32_t *far, uint8_t *keep,
                      int32_t *cnt, hipStream_t s) {
    ArcSrc a{};
    a.col = c.col;
    a.w = c.w;
    a.pk = c.pk;
    a.cb = c.cb;
    a.cmask = c.cb >= 32 ? 0xffffffffu : ((1u << c.cb) - 1u);
    const int grid = (pl.ntasks + kWavesPerBlock - 1) / kWavesPerBlock;
    if (grid < 1) return;
    if (c.pk)
        hipLaunchKernelGGL(k_core_mark<1>, dim3(grid), dim3(kBlock), 0, s, pl.tasks, pl.ntasks, c.rp, a,
                           (const uint32_t *)near, (const uint32_t *)far, keep, cnt);
    else
        hipLaunchKernelGGL(k_core_mark<2>, dim3(grid), dim3(kBlock), 0, s, pl.tasks, pl.ntasks, c.rp, a,
                           (const uint32_t *)near, (const uint32_t *)far, keep, cnt);
}

void launch_core_zero(int32_t *cnt, int n, hipStream_t s) {
    hipLaunchKernelGGL(k_core_zero, dim3((n + 255) / 256), dim3(256), 0, s, cnt, n);
}

void launch_core_hub(const int32_t *bound, int n, int32_t *out, hipStream_t s) {
    hipLaunchKernelGGL(k_core_hub, dim3((n + 255) / 256), dim3(256), 0, s, bound, n, out);
}

void launch_core_compact(int32_t n, const Csr &c, const uint8_t *keep, const Csr &out, hipStream_t s) {
    hipLaunchKernelGGL(k_core_compact, dim3((n + kWavesPerBlock - 1) / kWavesPerBlock), dim3(kBlock), 0, s, n,
                       c, keep, out);
}

}  // namespace mfbc
