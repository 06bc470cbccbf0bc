// Fixpoints in which every arc acts alike (hop levels on any graph; every
// algebra on a graph whose weights are all 1): an entry improves once, in the
// product that first reaches it, so a frontier row is a 64-bit mask per column
// group instead of 64 values, a product is the OR of the masks of the active
// in-neighbours, and the value is a function of the product's number.
//
// Layout: W groups (1, 2 or 4: 64, 128 or 256 columns) side by side,
// [q][v][W] words, so an arc gathers 8 W bytes where the value form gathers
// 256 W.  The number of the product that reached an entry is kept in binary,
// one mask plane per bit ([bit][q][v][W]): a newly reached entry is or-ed into
// the planes of the bits of j, and the export puts the numbers together.  The
// planes take the place of T (at most 31 x 8 B against 256 B per vertex and
// group) and only those the running j needs are cleared.
//
// A lane takes one arc: it tests the source's activity bit, gathers its masks
// and ors them into its row's words in LDS; then a lane takes one row and
// finishes it.  Bound by the scattered mask gathers (32 B of a 128-B line at
// W = 4) and, where nearly every arc is active, the LDS atomics of rows.
// 256 hop-level columns on R-MAT scale 19 (15.6 M arcs), ms: the products 4.95
// in the value form, 0.83 here (0.2 the densest); fill and export 0.46 / 0.22;
// the call 5.67 / 1.15.
#include <algorithm>

#include "products.h"

namespace mfbc {
namespace {

struct BitArgs {
    const Task *tasks;
    const Hub *hubs;
    int ntasks, nhubs, n, nwords, nq, j;
    const uint8_t *owner;        // row of each arc within its task
    const uint32_t *arc;         // packed arcs or columns
    uint32_t cmask;
    const uint32_t *bits;        // activity of F_{j-1}, one plane per q
    uint32_t *bits_n;
    const unsigned long long *f; // F_{j-1}, F_j, reached
    unsigned long long *f_n, *seen;
    unsigned long long *level;   // planes of `plane` words each
    size_t plane;
    unsigned long long *hub;     // [q][hub][W] OR of the slices, zero between products
    unsigned long long *ctr;
    const unsigned long long *prev_ctr;
    uint32_t *clear_bits;
    unsigned long long *clear_ctr;
    uint32_t *next_bits;         // no split rows: F_{j+1}'s bitmaps and counters (close_product)
    unsigned long long *next_ctr;
    const int64_t *rp;
};

template <int W>
struct Words {
    unsigned long long w[W];
};

template <int W>
__device__ __forceinline__ Words<W> load_words(const unsigned long long *p) {
    Words<W> r;
    if constexpr (W == 1) {
        r.w[0] = p[0];
    } else {
#pragma unroll
        for (int k = 0; k < W; k += 2) {
            const ulonglong2 x = *(const ulonglong2 *)(p + k);
            r.w[k] = x.x;
            r.w[k + 1] = x.y;
        }
    }
    return r;
}

template <int W>
__device__ __forceinline__ void store_words(unsigned long long *p, const Words<W> &r) {
    if constexpr (W == 1) {
        p[0] = r.w[0];
    } else {
#pragma unroll
        for (int k = 0; k < W; k += 2) *(ulonglong2 *)(p + k) = make_ulonglong2(r.w[k], r.w[k + 1]);
    }
}

// Row v given the OR `a` of its candidates: whether it joins the next frontier.
template <int W>
__device__ __forceinline__ bool finish_row(const BitArgs &a, int q, int v, const Words<W> &c,
                                           unsigned &produced, unsigned &outs) {
    unsigned long long any = 0;
#pragma unroll
    for (int k = 0; k < W; k++) {
        any |= c.w[k];
        outs += __popcll(c.w[k]);
    }
    if (!any) return false;
    const size_t at = ((size_t)q * a.n + v) * W;
    Words<W> s = load_words<W>(a.seen + at), x;
    any = 0;
#pragma unroll
    for (int k = 0; k < W; k++) {
        x.w[k] = c.w[k] & ~s.w[k];
        s.w[k] |= x.w[k];
        any |= x.w[k];
        produced += __popcll(x.w[k]);
    }
    if (!any) return false;
    store_words<W>(a.seen + at, s);
    store_words<W>(a.f_n + at, x);
    for (int b = 0; (a.j >> b) != 0; b++) {
        if (!((a.j >> b) & 1)) continue;
        unsigned long long *p = a.level + (size_t)b * a.plane + at;
        Words<W> l = load_words<W>(p);
#pragma unroll
        for (int k = 0; k < W; k++) l.w[k] |= x.w[k];
        store_words<W>(p, l);
    }
    return true;
}

__device__ __forceinline__ unsigned long long wave_add(unsigned x) {
    unsigned long long t = x;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off, kWave);
    return t;
}

__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int W, bool C>
__global__ __launch_bounds__(kBlock) void k_bits_pull(BitArgs a) {
    __shared__ unsigned long long s_acc[kWavesPerBlock][kWave * W];
    if (!live_prev(a.prev_ctr)) {
        if constexpr (C) close_skipped(a.next_ctr);
        return;
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = uni((int)(threadIdx.x >> 6));
    const int wid = blockIdx.x * kWavesPerBlock + wv;
    const int q = wid / a.ntasks;
    unsigned produced = 0, outs = 0;
    if (q < a.nq) {
        const Task *tp = a.tasks + (wid - q * a.ntasks);
        const int v0 = uni(tp->v0), v1 = uni(tp->v1), hub = uni(tp->hub);
        const int64_t e0 = uni64(tp->e0), e1 = uni64(tp->e1);
        const uint32_t *bits = a.bits + (size_t)q * a.nwords;
        const unsigned long long *f = a.f + (size_t)q * a.n * W;
        unsigned long long *acc = s_acc[wv];
        Words<W> own;
#pragma unroll
        for (int k = 0; k < W; k++) {
            own.w[k] = 0ull;
            acc[lane * W + k] = 0ull;
        }
        wave_sync_lds();
        for (int64_t e = e0 + lane; e < e1; e += kWave) {
            const uint32_t u = a.arc[e] & a.cmask;
            const int o = a.owner[e];
            if (!((bits[u >> 5] >> (u & 31)) & 1u)) continue;
            const Words<W> m = load_words<W>(f + (size_t)u * W);
#pragma unroll
            for (int k = 0; k < W; k++) {
                if (hub >= 0) own.w[k] |= m.w[k];
                else if (m.w[k]) atomicOr(acc + o * W + k, m.w[k]);
            }
        }
        if (hub >= 0) {
#pragma unroll
            for (int k = 0; k < W; k++) {
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) own.w[k] |= __shfl_xor(own.w[k], off, kWave);
                if (lane == 0 && own.w[k]) atomicOr(a.hub + ((size_t)q * a.nhubs + hub) * W + k, own.w[k]);
            }
        } else {
            wave_sync_lds();
            bool on = false;
            if (v0 + lane < v1) {
                Words<W> c;
#pragma unroll
                for (int k = 0; k < W; k++) c.w[k] = acc[lane * W + k];
                on = finish_row<W>(a, q, v0 + lane, c, produced, outs);
            }
            const uint64_t run = ballot(on);
            if (lane == 0 && run) or_run_bits(a.bits_n + (size_t)q * a.nwords, v0, run);
        }
    }
    unsigned long long nv = 0, na = 0;
    if constexpr (C) close_product(a.bits, a.next_bits, a.nwords, a.nq, a.rp, a.next_ctr, nv, na);
    flush_counts(wave_add(produced), wave_add(outs), nv, na, a.ctr);
}

// The split rows, one thread each; also clears F_{j-1}'s bitmaps (counting its
// vertices and their arcs) and the counters of product j+1.
template <int W>
__global__ __launch_bounds__(kBlock) void k_bits_merge(BitArgs a) {
    const int gtid = blockIdx.x * kBlock + threadIdx.x;
    if (!live_prev(a.prev_ctr)) {
        if (gtid < 4 * kCounterSlots) a.clear_ctr[gtid] = 0ull;
        return;
    }
    unsigned long long nv = 0, na = 0;
    clear_and_count(a.clear_bits, a.nwords, a.nq, a.rp, nv, na);
    if (gtid < 4 * kCounterSlots) a.clear_ctr[gtid] = 0ull;
    unsigned produced = 0, outs = 0;
    for (int i = gtid; i < a.nq * a.nhubs; i += gridDim.x * kBlock) {
        const int q = i / a.nhubs, v = a.hubs[i - q * a.nhubs].v;
        unsigned long long *p = a.hub + (size_t)i * W;
        const Words<W> c = load_words<W>(p);
        Words<W> z;
#pragma unroll
        for (int k = 0; k < W; k++) z.w[k] = 0ull;
        store_words<W>(p, z);
        if (finish_row<W>(a, q, v, c, produced, outs))
            atomicOr(a.bits_n + (size_t)q * a.nwords + (v >> 5), 1u << (v & 31));
    }
    flush_counts(wave_add(produced), wave_add(outs), nv, na, a.ctr);
}

__global__ void k_bits_zero(unsigned long long *p, size_t count) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) p[i] = 0ull;
}

// Nothing reached, no frontier, counters and hub words at zero.
__global__ void k_bits_init(unsigned long long *seen, size_t nseen, uint32_t *ab0, uint32_t *ab1, uint32_t *ab2, size_t nab,
                            unsigned long long *hub, size_t nhub, unsigned long long *ctr, int nctr) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const size_t t0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (size_t i = t0; i < nseen; i += stride) seen[i] = 0ull;
    for (size_t i = t0; i < nab; i += stride) {
        ab0[i] = 0u;
        ab1[i] = 0u;
        ab2[i] = 0u;
    }
    for (size_t i = t0; i < nhub; i += stride) hub[i] = 0ull;
    for (size_t i = t0; i < (size_t)nctr; i += stride) ctr[i] = 0ull;
}

// Seeds (launch_seed): the sources' rows of the first frontier start empty,
// then each column reaches its source.
template <int W>
struct BitSeed {
    static constexpr int kGroups = W;
    int n, nwords;
    unsigned long long *f, *seen;
    uint32_t *abits;
    __device__ void row(int v, int q, int lane) const {
        if (lane < W) f[((size_t)q * n + v) * W + lane] = 0ull;
    }
    __device__ void entry(int v, int c) const {
        const int q = c / (W * kWave), k = (c / kWave) % W;
        const size_t at = ((size_t)q * n + v) * W + k;
        const unsigned long long m = 1ull << (c % kWave);
        atomicOr(f + at, m);
        atomicOr(seen + at, m);
        atomicOr(abits + (size_t)q * nwords + (v >> 5), 1u << (v & 31));
    }
};

// Values of 64 caller vertices (one per lane) for the wave's 16 columns of
// group cg: the bits of the product number from `planes` words per vertex.
// V(level): the algebra's value, `far` where nothing reached.
template <int W, class V>
__global__ __launch_bounds__(kBlock) void k_bits_export(const unsigned long long *seen,
                                                        const unsigned long long *level, size_t plane,
                                                        int planes, int n, int nb, const int32_t *perm,
                                                        typename V::T *out) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = uni((int)(threadIdx.x >> 6));
    const int v = blockIdx.x * kWave + lane, cg = blockIdx.y;
    if (v >= n) return;
    const int d = perm ? perm[v] : v;
    const size_t at = ((size_t)(cg / W) * n + d) * W + cg % W;
    const int c0 = wv * 16;
    const uint32_t s = (uint32_t)(seen[at] >> c0) & 0xffffu;
    uint32_t x[16];
#pragma unroll
    for (int i = 0; i < 16; i++) x[i] = 0u;
    for (int b = 0; b < planes; b++) {
        const uint32_t w = (uint32_t)(level[(size_t)b * plane + at] >> c0);
#pragma unroll
        for (int i = 0; i < 16; i++) x[i] |= ((w >> i) & 1u) << b;
    }
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const int c = cg * kWave + c0 + i;
        if (c < nb) out[(size_t)c * n + v] = (s >> i) & 1u ? V::at(x[i]) : V::far();
    }
}

struct HopLevel {            // sssp on unit weights, bfs
    using T = int32_t;
    __device__ static T at(uint32_t j) { return (int32_t)j; }
    __device__ static T far() { return kInf; }
};
struct UnitWidth {           // widest: the source's own width is unbounded
    using T = int32_t;
    __device__ static T at(uint32_t j) { return j ? 1 : kInf; }
    __device__ static T far() { return 0; }
};
struct UnitSum {             // resist: j additions of 1 / 1
    using T = float;
    __device__ static T at(uint32_t j) { return (float)j; }
    __device__ static T far() { return __builtin_inff(); }
};

int grid_for(size_t work, int per, size_t cap) {
    return (int)std::max<size_t>(1, std::min<size_t>((work + per - 1) / per, cap));
}

// Groups side by side for a batch: one pass over the arcs serves them all.
// The workspace holds one group or an even number of them.
int bits_width(int ncg) {
    if (ncg <= 1) return 1;
    return ((ncg + 1) & ~1) % 4 == 0 ? 4 : 2;
}

BitArgs bit_args(mfbc_graph *g, int ncg, int j) {
    Workspace &ws = g->ws;
    const View &vw = g->full;
    const int W = bits_width(ncg), b = (j - 1) & 1;
    BitArgs a{};
    a.tasks = vw.plan_in.tasks;
    a.hubs = vw.plan_in.hubs;
    a.ntasks = vw.plan_in.ntasks;
    a.nhubs = vw.plan_in.nhubs;
    a.n = g->n;
    a.nwords = (g->n + 31) / 32;
    a.nq = (ncg + W - 1) / W;
    a.j = j;
    a.owner = vw.plan_in.owner;
    a.arc = vw.in.pk ? vw.in.pk : (const uint32_t *)vw.in.col;
    a.cmask = vw.in.pk && vw.in.cb < 32 ? (1u << vw.in.cb) - 1u : 0xffffffffu;
    a.bits = ws.abits[(j - 1) % 3];
    a.bits_n = ws.abits[j % 3];
    a.f = (const unsigned long long *)ws.fbits[b];
    a.f_n = (unsigned long long *)ws.fbits[b ^ 1];
    a.seen = (unsigned long long *)ws.lam;       // 8 B per vertex and group, as the masks
    a.level = (unsigned long long *)ws.tdist;
    a.plane = (size_t)a.nq * g->n * W;
    a.hub = (unsigned long long *)ws.pd;
    a.ctr = ws.counters + (size_t)(j % kCounterRing) * 4 * kCounterSlots;
    a.prev_ctr = j > 1 ? ws.counters + (size_t)((j - 1) % kCounterRing) * 4 * kCounterSlots : nullptr;
    a.clear_bits = ws.abits[(j - 1) % 3];
    a.clear_ctr = ws.counters + (size_t)((j + 1) % kCounterRing) * 4 * kCounterSlots;
    if (a.nhubs == 0) {
        a.next_bits = ws.abits[(j + 1) % 3];
        a.next_ctr = a.clear_ctr;
    }
    a.rp = vw.in.rp;
    return a;
}

template <int W>
void bits_init(const BitArgs &a, mfbc_graph *g, int ncg, int nb, const int32_t *d_sources, hipStream_t s) {
    Workspace &ws = g->ws;
    hipLaunchKernelGGL(k_bits_init, dim3(grid_for(a.plane, 256, 8192)), dim3(256), 0, s, a.seen, a.plane,
                       ws.abits[0], ws.abits[1], ws.abits[2], (size_t)a.nq * a.nwords, a.hub,
                       (size_t)a.nq * a.nhubs * W, ws.counters, (int)kRingWords);
    const BitSeed<W> seed{g->n, a.nwords, (unsigned long long *)ws.fbits[0], a.seen, ws.abits[0]};
    launch_seed(g, seed, ncg, nb, d_sources, s);
}

template <int W>
void bits_product(const BitArgs &a, hipStream_t s, hipEvent_t *ev) {
    if (ev) (void)hipEventRecord(ev[0], s);
    const int grid = grid_for((size_t)a.ntasks * a.nq, kWavesPerBlock, 0x7fffffff);
    if (a.next_bits) hipLaunchKernelGGL((k_bits_pull<W, true>), dim3(grid), dim3(kBlock), 0, s, a);
    else hipLaunchKernelGGL((k_bits_pull<W, false>), dim3(grid), dim3(kBlock), 0, s, a);
    if (ev) (void)hipEventRecord(ev[1], s);
    const size_t work = std::max((size_t)a.nhubs * a.nq, (size_t)a.nwords);
    if (a.nhubs)
        hipLaunchKernelGGL(k_bits_merge<W>, dim3(grid_for(work, kBlock, 1024)), dim3(kBlock), 0, s, a);
    if (ev && ev[2]) (void)hipEventRecord(ev[2], s);
}

template <int W>
void bits_export(const BitArgs &a, mfbc_graph *g, int op, int ncg, int nb, int planes, void *out, hipStream_t s) {
    const dim3 grid((g->n + kWave - 1) / kWave, ncg);
    const int32_t *perm = g->perm;
    if (op == MFBC_OP_RESIST)
        hipLaunchKernelGGL((k_bits_export<W, UnitSum>), grid, dim3(kBlock), 0, s, a.seen, a.level, a.plane, planes,
                           g->n, nb, perm, (float *)out);
    else if (op == MFBC_OP_WIDEST)
        hipLaunchKernelGGL((k_bits_export<W, UnitWidth>), grid, dim3(kBlock), 0, s, a.seen, a.level, a.plane,
                           planes, g->n, nb, perm, (int32_t *)out);
    else
        hipLaunchKernelGGL((k_bits_export<W, HopLevel>), grid, dim3(kBlock), 0, s, a.seen, a.level, a.plane,
                           planes, g->n, nb, perm, (int32_t *)out);
}

__global__ __launch_bounds__(kBlock) void k_plan_owner(const Task *tasks, int ntasks, const int64_t *rp,
                                                       uint8_t *owner) {
    const int lane = threadIdx.x & (kWave - 1);
    const int t = blockIdx.x * kWavesPerBlock + uni((int)(threadIdx.x >> 6));
    if (t >= ntasks) return;
    const Task *tp = tasks + t;
    const int v0 = uni(tp->v0), v1 = uni(tp->v1);
    if (uni(tp->hub) >= 0) {
        const int64_t e1 = uni64(tp->e1);
        for (int64_t e = uni64(tp->e0) + lane; e < e1; e += kWave) owner[e] = 0;
        return;
    }
    for (int v = v0; v < v1; v++) {
        const int64_t e1 = rp[v + 1];
        for (int64_t e = rp[v] + lane; e < e1; e += kWave) owner[e] = (uint8_t)(v - v0);
    }
}

}  // namespace

void launch_plan_owner(const Csr &c, const Plan &pl, hipStream_t s) {
    const int grid = (pl.ntasks + kWavesPerBlock - 1) / kWavesPerBlock;
    if (grid > 0) hipLaunchKernelGGL(k_plan_owner, dim3(grid), dim3(kBlock), 0, s, pl.tasks, pl.ntasks, c.rp, pl.owner);
}

// Every arc acts alike: hop levels, and every algebra on unit weights (sums of
// 1/1 are exact while a path's arcs stay below 2^24).
bool bits_fit(const mfbc_graph *g, int op) {
    if (op == MFBC_OP_BFS) return true;
    return g->maxw == 1 && (op != MFBC_OP_RESIST || g->n < (1 << 24));
}

void launch_bits_init(mfbc_graph *g, int ncg, int nb, const int32_t *d_sources, hipStream_t s) {
    const BitArgs a = bit_args(g, ncg, 1);
    switch (bits_width(ncg)) {
        case 1: bits_init<1>(a, g, ncg, nb, d_sources, s); break;
        case 2: bits_init<2>(a, g, ncg, nb, d_sources, s); break;
        default: bits_init<4>(a, g, ncg, nb, d_sources, s); break;
    }
}

// Clears the planes of bits [from, to) of the product number.
void launch_bits_planes(mfbc_graph *g, int ncg, int from, int to, hipStream_t s) {
    if (to <= from) return;
    const BitArgs a = bit_args(g, ncg, 1);
    const size_t words = (size_t)(to - from) * a.plane;
    hipLaunchKernelGGL(k_bits_zero, dim3(grid_for(words, 256, 8192)), dim3(256), 0, s,
                       a.level + (size_t)from * a.plane, words);
}

void launch_bits_product(mfbc_graph *g, int ncg, int j, hipStream_t s, hipEvent_t *ev) {
    const BitArgs a = bit_args(g, ncg, j);
    switch (bits_width(ncg)) {
        case 1: bits_product<1>(a, s, ev); break;
        case 2: bits_product<2>(a, s, ev); break;
        default: bits_product<4>(a, s, ev); break;
    }
}

void launch_bits_export(mfbc_graph *g, int op, int ncg, int nb, int planes, void *out, hipStream_t s) {
    const BitArgs a = bit_args(g, ncg, 1);
    switch (bits_width(ncg)) {
        case 1: bits_export<1>(a, g, op, ncg, nb, planes, out, s); break;
        case 2: bits_export<2>(a, g, op, ncg, nb, planes, out, s); break;
        default: bits_export<4>(a, g, op, ncg, nb, planes, out, s); break;
    }
}

}  // namespace mfbc
