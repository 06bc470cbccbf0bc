// Distances and path counts (MFBF, Algorithm 1) and shortest distances (the
// min, a + w fixpoint) of a batch in 16 bits an entry, on every arc of the
// graph, and for centrality on its shortest-path core.  Same products,
// frontiers and results as the 32-bit forms in products.h and monoid.hip; three
// things make them cheaper (the first alone on a core).
//
// 1. A frontier entry of product j has j arcs, so its weight is at most j times
//    the largest weight: while that leaves room, weight and multiplicity share
//    16 bits, (weight << mb) | m with mb as large as the product allows, and
//    Q words a lane hold 2 Q column groups (128 or 256 columns): an arc's
//    gather moves 256 Q bytes for 128 Q columns, half of the 32-bit form's, and
//    with Q = 2 one instruction serves 256 columns.  m = 2^mb - 1 means "or
//    more": the value is in the binary64 array, and sums that reach it are
//    taken again in binary64, over the row's arcs in order.  The encoding is
//    exact.  A call whose frontier outlives the products that fit
//    (quad_products) goes on in 32 bits from there (k_quad_widen).  T in this layout is what the paired counting
//    product of a centrality call reads, so no copy of it is made.  T's
//    multiplicities are kept the same way, 16 bits with the binary64 array behind
//    those that do not fit: a kept entry writes 6 bytes where it wrote 12, and
//    the backward half reads 2 for 8 (centrality of 256 sources on weighted R-MAT
//    scale 20: 12.5 ms before, 9.6 so).
//
// 2. An arc u -> v can change v only if F(u) + w <= T(v) in some column (< for
//    distances alone).  Columns differ mostly by how far their source is from
//    the rest of the graph, so the test is made against bounds relative to an
//    offset h of each column, the distance from its source to the landmark of
//    highest degree (core.hip):
//        min over columns of (F(u) - h) + w <= max over columns of (T(v) - h)
//    with the left minimum kept per frontier row (16 bits, `lo`) and the right
//    maximum per vertex (`hi`, columns whose frontier has died out left out).
//    Any offsets are sound; these leave 29% of the gathers on weighted R-MAT
//    graphs and 23% on uniform ones of degree 256.  On a core nearly every arc
//    passes and rows are short, so no bounds are kept (centrality of all sources
//    of a uniform graph of 1,024 vertices, degree 8: 1.32 ms with, 1.03 without;
//    uniform, degree 60, n = 10,000, 900 sources: 3.5 / 2.6).
//
// 3. `lo` is also the activity test, so that a chunk of arcs makes one gather
//    of 16-bit words where the 32-bit forms gather bitmap words.
#include <algorithm>

#include "products.h"

namespace mfbc {
namespace {

constexpr uint32_t kNone16 = 0xffffu;        // an absent entry, an unreached T
constexpr uint32_t kNone32 = 0xffffffffu;    // two of them
constexpr int kLoBias = 16384;               // lo = bound + kLoBias, 0: below every code
constexpr uint32_t kLoOff = 0xffffu;         // not in the frontier
constexpr int kLiveCopies = 32;              // of the live-column masks, by workgroup: one copy
                                             // cost small graphs 20 to 40 us a product in
                                             // atomics on the same words

typedef unsigned short us2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ us2 as2(uint32_t x) { return __builtin_bit_cast(us2, x); }
__device__ __forceinline__ uint32_t as1(us2 x) { return __builtin_bit_cast(uint32_t, x); }
__device__ __forceinline__ us2 both(uint32_t x) { return as2(x | (x << 16)); }
__device__ __forceinline__ uint32_t half_of(uint32_t x, int h) { return h ? x >> 16 : x & 0xffffu; }

struct QuadArgs {
    const Task *tasks;
    const Hub *hubs;
    int ntasks, nhubs, nslots, ncg, n, nwords, nq;
    const int64_t *rp;
    ArcSrc arcs;
    const uint8_t *owner;        // row of each arc within its task
    const uint32_t *f;           // F_{j-1}: [q][n][64][Q] words of two entries
    uint32_t *f_n;               // F_j
    uint32_t *t;                 // T, same layout
    const uint16_t *lo;          // [q][n] of F_{j-1}, F_j, and those to clear (F_{j+1}'s)
    uint16_t *lo_n, *lo_clear;
    int32_t *hi;                 // [q][n]
    const int32_t *off;          // h of each column
    const unsigned long long *live;   // columns with entries in F_{j-1}, F_j, F_{j+1}:
                                 // [ncg][kLiveCopies], the masks' OR
    unsigned long long *live_n, *live_clear;
    uint32_t *done;              // nullable: rows whose T is final in every column, [q][nwords]
    const int32_t *src;          // column -> source vertex, -1 = padding
    const uint32_t *bits;        // activity bitmaps, [q][nwords]
    uint32_t *bits_n, *next_bits;
    int32_t *pd;                 // hub partials [cg][slot][64]
    double *pm;
    unsigned long long *ctr, *next_ctr;
    const unsigned long long *prev_ctr;
    // multiplicities
    int mb, mbn;                 // bits of m in F_{j-1} and F_j
    uint32_t *sig;               // multiplicities of T, laid out as T: 16 bits where they fit,
    double *tsig;                // else kSig16Far and the value here, [cg][n][64]
    const double *fsig;
    double *fsig_n;
    int32_t *flags;
};

// Largest (smallest) value over the wave, in every lane.
template <bool MAX>
__device__ __forceinline__ int wave_extreme(int x) {
    const int id = MAX ? INT32_MIN : INT32_MAX;
    auto op = [](int a, int b) { return MAX ? (a > b ? a : b) : (a < b ? a : b); };
    x = op(x, __builtin_amdgcn_update_dpp(id, x, 0x111, 0xf, 0xf, false));    // row_shr 1, 2, 4, 8
    x = op(x, __builtin_amdgcn_update_dpp(id, x, 0x112, 0xf, 0xf, false));
    x = op(x, __builtin_amdgcn_update_dpp(id, x, 0x114, 0xf, 0xf, false));
    x = op(x, __builtin_amdgcn_update_dpp(id, x, 0x118, 0xf, 0xf, false));
    x = op(x, __builtin_amdgcn_update_dpp(id, x, 0x142, 0xa, 0xf, false));    // row_bcast 15, 31
    x = op(x, __builtin_amdgcn_update_dpp(id, x, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(x, 63);
}

// OR of the values of lanes 0..31 (lanes 32..63 hold the same ones again).
__device__ __forceinline__ uint64_t or_copies(uint64_t x) {
    int w[2] = {(int)(uint32_t)x, (int)(uint32_t)(x >> 32)};
#pragma unroll
    for (int k = 0; k < 2; k++) {
        w[k] |= __builtin_amdgcn_update_dpp(0, w[k], 0x111, 0xf, 0xf, false);
        w[k] |= __builtin_amdgcn_update_dpp(0, w[k], 0x112, 0xf, 0xf, false);
        w[k] |= __builtin_amdgcn_update_dpp(0, w[k], 0x114, 0xf, 0xf, false);
        w[k] |= __builtin_amdgcn_update_dpp(0, w[k], 0x118, 0xf, 0xf, false);
        w[k] |= __builtin_amdgcn_update_dpp(0, w[k], 0x142, 0xa, 0xf, false);
        w[k] = rdlane(w[k], 31);
    }
    return ((uint64_t)(uint32_t)w[1] << 32) | (uint32_t)w[0];
}

template <int Q>
struct Lane {
    uint32_t w[Q];
};
template <int Q>
__device__ __forceinline__ Lane<Q> load_lane(const uint32_t *p, size_t row, int lane) {
    Lane<Q> r;
    if constexpr (Q == 1) {
        r.w[0] = p[row * kWave + lane];
    } else {
        const uint2 x = ((const uint2 *)p)[row * kWave + lane];
        r.w[0] = x.x;
        r.w[1] = x.y;
    }
    return r;
}
template <int Q>
__device__ __forceinline__ void store_lane(uint32_t *p, size_t row, int lane, const Lane<Q> &r) {
    if constexpr (Q == 1) p[row * kWave + lane] = r.w[0];
    else ((uint2 *)p)[row * kWave + lane] = make_uint2(r.w[0], r.w[1]);
}

// One wave's product: COUNT carries multiplicities (MFBF), else distances only.
// B: arcs are tested against the bounds; without (on a core) the activity bitmap
// is the test and no bound, offset or live-column mask is kept.
template <int AM, int Q, bool COUNT, bool B>
struct QuadPull {
    static constexpr int G = 2 * Q;              // column groups per lane
    static constexpr int U = Q == 1 ? 8 : 4;     // active arcs per batch
    // Without weights T(v) is final once set: a row that every column has reached
    // takes no part in later products, and a run of such rows reads no arcs
    // (`done`; centrality of 2,048 sources on R-MAT scale 16: 13.0 ms without,
    // 12.0 with; 600 sources at scale 18: 14.7 / 13.2; uniform n = 20,000 of
    // degree 100: 3.4 / 3.2).
    static constexpr bool D = AM == 0 && COUNT && !B;
    const QuadArgs a;            // by value, for the same reason as in task()
    const int q, lane;
    const size_t n, row0;
    unsigned long long produced = 0, outs = 0;
    uint64_t any[G];                             // lanes of each group that produced entries
    int off[G];
    uint32_t live = 0;                           // bit g: this lane's column of group g is live (B), in use (D)
    bool whole = false;                          // the row last finished: reached by every column

    __device__ __forceinline__ QuadPull(const QuadArgs &a_, int q_)
        : a(a_), q(q_), lane(threadIdx.x & (kWave - 1)), n((size_t)a_.n), row0((size_t)q_ * a_.n) {
#pragma unroll
        for (int g = 0; g < G; g++) {
            any[g] = 0;
            const int cg = q * G + g;
            off[g] = 0;
            if constexpr (D) live |= (uint32_t)(cg < a.ncg && a.src[cg * kWave + lane] >= 0) << g;
            if constexpr (!B) continue;
            off[g] = cg < a.ncg ? a.off[cg * kWave + lane] : 0;
            if (cg < a.ncg) live |= (uint32_t)((or_copies(a.live[cg * kLiveCopies + (lane & (kLiveCopies - 1))]) >> lane) & 1ull) << g;
        }
    }
    __device__ __forceinline__ size_t at(int g, int v) const {
        return ((size_t)(q * G + g) * n + (size_t)v) * kWave + lane;
    }
    __device__ __forceinline__ bool pass(uint32_t x, int w, int thr) const {
        if (x == kLoOff) return false;
        const int least = (int)x - kLoBias + w;
        return x == 0u || (COUNT ? least <= thr : least < thr);
    }
    __device__ __forceinline__ void fold(Lane<Q> &acc, const Lane<Q> &r, int w) const {
        const int sh = COUNT ? a.mb : 0;
        const us2 ww = both((uint32_t)w << sh);
#pragma unroll
        for (int k = 0; k < Q; k++) {
            const us2 c = __builtin_elementwise_add_sat(as2(r.w[k]), ww);   // an absent entry stays one
            const us2 x = as2(acc.w[k]);
            const us2 mn = __builtin_elementwise_min(x, c);
            if constexpr (!COUNT) {
                acc.w[k] = as1(mn);
            } else {
                // equal weights: the multiplicities' sum, held at 2^mb - 1
                const us2 mm = both((1u << a.mb) - 1u), bits = both((uint32_t)a.mb);
                const us2 mx = __builtin_elementwise_max(x, c);
                const us2 base = mn & ~mm;
                const us2 e = mx - base;
                const us2 tie = __builtin_elementwise_sub_sat(both(1u), e >> bits);
                const us2 m = __builtin_elementwise_min((us2)((mn & mm) + tie * e), mm);
                acc.w[k] = as1(base | m);
            }
        }
    }
    // Weights and multiplicities of the candidates in `acc` (weight kNone16:
    // none); whether one that T keeps is saturated, so that the row's arcs have
    // to be summed in binary64 (walk).
    __device__ __forceinline__ bool expand(const Lane<Q> &acc, const Lane<Q> &own, uint32_t (&d)[G],
                                           double (&m)[G]) const {
        bool some = false;
        const uint32_t mm = COUNT ? (1u << a.mb) - 1u : 0u;
#pragma unroll
        for (int g = 0; g < G; g++) {
            const uint32_t x = half_of(acc.w[g >> 1], g & 1);
            d[g] = !COUNT || x == kNone16 ? x : x >> a.mb;
            m[g] = COUNT ? (double)(x & mm) : 0.0;
            some |= COUNT && x != kNone16 && (x & mm) == mm && d[g] <= half_of(own.w[g >> 1], g & 1);
        }
        return COUNT && ballot(some) != 0ull;
    }
    // The same from the arcs [ea, eb) of the row, in order, in binary64 (rows
    // with a saturated entry: 0.1% of those of weighted R-MAT graphs).
    __device__ __forceinline__ void walk(int64_t ea, int64_t eb, uint32_t (&d)[G], double (&m)[G]) const {
        const uint32_t mm = (1u << a.mb) - 1u;
#pragma unroll
        for (int g = 0; g < G; g++) {
            d[g] = kNone16;
            m[g] = 0.0;
        }
        for (int64_t e = ea; e < eb; e += kWave) {
            const int64_t my = e + lane;
            int u = 0, wt = 1;
            bool act = false;
            if (my < eb) {
                load_arc<AM>(a.arcs, my, u, wt);
                if constexpr (B) act = a.lo[row0 + (size_t)(uint32_t)u] != kLoOff;
                else act = (a.bits[(size_t)q * a.nwords + (u >> 5)] >> (u & 31)) & 1u;
            }
            uint64_t am = ballot(act);
            while (am) {
                const int j = __builtin_ctzll(am);
                am &= am - 1;
                const int uj = rdlane(u, j), wj = AM ? rdlane(wt, j) : 1;
                const Lane<Q> r = load_lane<Q>(a.f, row0 + (size_t)(uint32_t)uj, lane);
#pragma unroll
                for (int g = 0; g < G; g++) {
                    const uint32_t x = half_of(r.w[g >> 1], g & 1);
                    const uint32_t c = (x >> a.mb) + (uint32_t)wj;
                    if (x != kNone16 && c <= d[g]) {
                        const double y = (x & mm) != mm ? (double)(x & mm) : a.fsig[at(g, uj)];
                        m[g] = c < d[g] ? y : m[g] + y;
                        d[g] = c;
                    }
                }
            }
        }
    }
    // T := T (+) G at v, the next frontier row and the bounds.
    __device__ __forceinline__ bool finish(int v, const uint32_t (&d)[G], const double (&m)[G], const Lane<Q> &own) {
        uint64_t hm = 0;
#pragma unroll
        for (int g = 0; g < G; g++) {
            const uint64_t h = ballot(d[g] != kNone16);
            outs += __popcll(h);
            hm |= h;
        }
        if (!hm) return false;
        Lane<Q> nt = own, nf, ns;
        if constexpr (COUNT && B) {
            // with bounds a third of the rows keep nothing (forward of 200 sources,
            // weighted R-MAT scale 18: 4.97 ms without this look, 4.75 with)
            bool some = false;
#pragma unroll
            for (int g = 0; g < G; g++) some |= d[g] <= half_of(own.w[g >> 1], g & 1) && d[g] != kNone16;
            if (!ballot(some)) return false;
        }
        if constexpr (COUNT) ns = load_lane<Q>(a.sig, row0 + (size_t)v, lane);
        int least = INT32_MAX, most = INT32_MIN;
        uint64_t kept = 0, open = 0;
#pragma unroll
        for (int k = 0; k < Q; k++) nf.w[k] = kNone32;
#pragma unroll
        for (int g = 0; g < G; g++) {
            const uint32_t t = half_of(own.w[g >> 1], g & 1);
            const bool keep = d[g] != kNone16 && (COUNT ? d[g] <= t : d[g] < t);
            const int sh = (g & 1) * 16;
            uint32_t tn = t;
            if (keep) {
                tn = d[g];
                uint32_t x = d[g];
                if constexpr (COUNT) {
                    const size_t i = at(g, v);
                    const uint32_t si = half_of(ns.w[g >> 1], g & 1);
                    double s = m[g];
                    if (d[g] == t) s += si != kSig16Far ? (double)si : a.tsig[i];
                    uint32_t sn = kSig16Far;
                    if (s < (double)kSig16Far) {
                        sn = (uint32_t)s;
                    } else {
                        a.tsig[i] = s;
                        if (__builtin_isinf(s)) a.flags[0] = 1;
                    }
                    ns.w[g >> 1] = (ns.w[g >> 1] & ~(0xffffu << sh)) | (sn << sh);
                    const uint32_t most_m = (1u << a.mbn) - 1u;
                    uint32_t mi = most_m;
                    if (m[g] < (double)most_m) mi = (uint32_t)m[g];
                    else a.fsig_n[i] = m[g];
                    x = (d[g] << a.mbn) | mi;
                }
                nt.w[g >> 1] = (nt.w[g >> 1] & ~(0xffffu << sh)) | (d[g] << sh);
                nf.w[g >> 1] = (nf.w[g >> 1] & ~(0xffffu << sh)) | (x << sh);
                const int r = (int)d[g] - off[g];
                if (B && r < least) least = r;
            }
            if (B && ((live >> g) & 1u)) {
                const int r = tn == kNone16 ? INT32_MAX : (int)tn - off[g];
                if (r > most) most = r;
            }
            const uint64_t b = ballot(keep);
            produced += __popcll(b);
            kept |= b;
            if constexpr (B) any[g] |= b;
            if constexpr (D) open |= ballot(((live >> g) & 1u) && tn == kNone16);
        }
        if constexpr (D) whole = open == 0;
        if (!kept) return false;
        store_lane<Q>(a.t, row0 + (size_t)v, lane, nt);
        if constexpr (COUNT) store_lane<Q>(a.sig, row0 + (size_t)v, lane, ns);
        store_lane<Q>(a.f_n, row0 + (size_t)v, lane, nf);
        if constexpr (!B) return true;
        least = wave_extreme<false>(least);
        most = wave_extreme<true>(most);
        if (lane == 0) {
            int code = least + kLoBias;
            code = code < 0 ? 0 : code > 65534 ? 65534 : code;
            a.lo_n[row0 + (size_t)v] = (uint16_t)code;
            a.hi[row0 + (size_t)v] = most;
        }
        return true;
    }
    __device__ __forceinline__ void task(int t) {
        const Task *tp = a.tasks + t;
        const int v0 = uni(tp->v0), v1 = uni(tp->v1), hub = uni(tp->hub), part = uni(tp->part);
        const int64_t e0 = uni64(tp->e0), e1 = uni64(tp->e1);
        const uint16_t *lo = B ? a.lo + row0 : nullptr;
        const uint32_t *bits = a.bits + (size_t)q * a.nwords;
        uint64_t closed = 0, full = 0;   // rows that are done, before and after
        if constexpr (D) {
            const uint32_t *dw = a.done + (size_t)q * a.nwords + (v0 >> 5);
            const int sh = v0 & 31, last = a.nwords - 1 - (v0 >> 5);
            const uint64_t w0 = uni((int)dw[0]) & 0xffffffffu, w1 = last > 0 ? uni((int)dw[1]) & 0xffffffffu : 0u;
            closed = (w0 | (w1 << 32)) >> sh;
            if (sh && last > 1) closed |= (uint64_t)(uint32_t)uni((int)dw[2]) << (64 - sh);
            const int rows = hub < 0 ? v1 - v0 : 1;
            if (!(~closed & (rows < kWave ? (1ull << rows) - 1ull : ~0ull))) return;
        }
        const int thr_l = B && v0 + lane < v1 ? a.hi[row0 + (size_t)(v0 + lane)] : INT32_MIN;
        int cur = -1;            // row (offset from v0) of the open reduction
        Lane<Q> acc, own;
#pragma unroll
        for (int k = 0; k < Q; k++) acc.w[k] = own.w[k] = kNone32;
        uint64_t run = 0, again = 0;     // rows in the next frontier; rows to walk
        auto close = [&]() __attribute__((always_inline)) {
            uint32_t d[G];
            double m[G];
            // (by value: two branches that or into one of two variables leave
            // both, and the kernel's arguments, in scratch memory)
            const bool walk_it = expand(acc, own, d, m);
            const bool joins = !walk_it && finish(v0 + cur, d, m, own);
            again |= (uint64_t)walk_it << cur;
            run |= (uint64_t)joins << cur;
            if constexpr (D) full |= (uint64_t)(joins && whole) << cur;
        };
        uint32_t rn0 = 0, rn1 = 1;
        int on0 = 0;
        if (e0 + lane < e1) {
            load_arc_raw<AM>(a.arcs, e0 + lane, rn0, rn1);
            on0 = a.owner[e0 + lane];
        }
        for (int64_t e = e0; e < e1; e += kWave) {
            const int64_t my = e + lane;
            int u, wt;
            decode_arc<AM>(a.arcs, rn0, rn1, u, wt);
            const int o = on0;
            uint32_t x = kLoOff;
            bool act = false;
            if (my < e1) {
                if constexpr (B) x = lo[(uint32_t)u];
                else act = (bits[u >> 5] >> (u & 31)) & 1u;
            }
            if (my + kWave < e1) {
                load_arc_raw<AM>(a.arcs, my + kWave, rn0, rn1);
                on0 = a.owner[my + kWave];
            }
            if constexpr (B) act = pass(x, wt, __shfl(thr_l, o, kWave));
            if constexpr (D) act = act && !((closed >> o) & 1ull);
            uint64_t am = ballot(act);
            int na = __popcll(am);
            while (na > 0) {
                int ow[U], wk[U];
                Lane<Q> rk[U], on[U];
                int prev = cur;
#pragma unroll
                for (int k = 0; k < U; k++) {
                    ow[k] = -1;
                    wk[k] = 0;
#pragma unroll
                    for (int c = 0; c < Q; c++) rk[k].w[c] = on[k].w[c] = kNone32;
                    if (k < na) {
                        const int j = __builtin_ctzll(am);
                        am &= ~(1ull << j);
                        wk[k] = AM ? rdlane(wt, j) : 1;
                        rk[k] = load_lane<Q>(a.f, row0 + (size_t)(uint32_t)rdlane(u, j), lane);
                        ow[k] = rdlane(o, j);
                        if (ow[k] != prev) on[k] = load_lane<Q>(a.t, row0 + (size_t)(v0 + ow[k]), lane);
                        prev = ow[k];
                    }
                }
                na -= U;
#pragma unroll
                for (int k = 0; k < U; k++) {
                    if (ow[k] >= 0) {
                        if (ow[k] != cur) {
                            if (cur >= 0) close();
                            cur = ow[k];
                            own = on[k];
#pragma unroll
                            for (int c = 0; c < Q; c++) acc.w[c] = kNone32;
                        }
                        fold(acc, rk[k], wk[k]);
                    }
                }
            }
        }
        if (hub < 0) {
            if (cur >= 0) close();
            while (COUNT && again) {
                const int o = __builtin_ctzll(again), v = v0 + o;
                again &= again - 1;
                uint32_t d[G];
                double m[G];
                walk(a.rp[v], a.rp[v + 1], d, m);
                if (finish(v, d, m, load_lane<Q>(a.t, row0 + (size_t)v, lane))) {
                    run |= 1ull << o;
                    if constexpr (D) full |= (uint64_t)whole << o;
                }
            }
            if (lane == 0 && run) or_run_bits(a.bits_n + (size_t)q * a.nwords, v0, run);
            if constexpr (D)
                if (lane == 0 && full) or_run_bits(a.done + (size_t)q * a.nwords, v0, full);
            return;
        }
        // a slice of a split row: its candidates, exact, for the merge (which skips
        // a row that is done, as its slices do)
        uint32_t d[G];
        double m[G];
        if (expand(acc, own, d, m)) walk(e0, e1, d, m);
#pragma unroll
        for (int g = 0; g < G; g++) {
            const int cg = q * G + g;
            if (cg >= a.ncg) continue;
            const size_t i = ((size_t)cg * a.nslots + part) * kWave + lane;
            a.pd[i] = (int)d[g];
            if constexpr (COUNT) a.pm[i] = m[g];
        }
    }
    __device__ __forceinline__ void merge(int h) {
        const Hub *hp = a.hubs + h;
        const int v = uni(hp->v), first = uni(hp->first), np = uni(hp->nparts);
        uint32_t *dw = a.done ? a.done + (size_t)q * a.nwords + (v >> 5) : nullptr;
        if (D && dw && ((uni((int)*dw) >> (v & 31)) & 1)) return;
        uint32_t d[G];
        double m[G];
#pragma unroll
        for (int g = 0; g < G; g++) {
            d[g] = kNone16;
            m[g] = 0.0;
        }
        // slices in flight: a row of 100 slices is a chain of its loads (path counts
        // of 200 sources at scale 18: 4.91 ms at four, 4.77 at eight, 4.79 at 12)
        constexpr int H = 8;
        for (int s0 = first; s0 < first + np; s0 += H) {
            uint32_t x[H][G];
            double y[H][G];
#pragma unroll
            for (int k = 0; k < H; k++)
#pragma unroll
                for (int g = 0; g < G; g++) {
                    const int cg = q * G + g;
                    x[k][g] = kNone16;
                    y[k][g] = 0.0;
                    if (s0 + k < first + np && cg < a.ncg) {
                        const size_t i = ((size_t)cg * a.nslots + s0 + k) * kWave + lane;
                        x[k][g] = (uint32_t)a.pd[i];
                        if constexpr (COUNT) y[k][g] = a.pm[i];
                    }
                }
#pragma unroll
            for (int k = 0; k < H; k++)
#pragma unroll
                for (int g = 0; g < G; g++) {
                    if (x[k][g] < d[g]) {
                        d[g] = x[k][g];
                        m[g] = y[k][g];
                    } else if (x[k][g] == d[g]) {
                        m[g] += y[k][g];
                    }
                }
        }
        const Lane<Q> own = load_lane<Q>(a.t, row0 + (size_t)v, lane);
        if (finish(v, d, m, own) && lane == 0) {
            atomicOr(a.bits_n + (size_t)q * a.nwords + (v >> 5), 1u << (v & 31));
            if (D && dw && whole) atomicOr(dw, 1u << (v & 31));
        }
    }
    // Columns that produced entries: an atomic where a bit looks new (a stale
    // word costs an atomic more).
    __device__ __forceinline__ void flush() const {
#pragma unroll
        for (int g = 0; g < G; g++) {
            const int cg = q * G + g;
            if (lane == g && cg < a.ncg && any[g]) {
                unsigned long long *p = a.live_n + cg * kLiveCopies + (blockIdx.x & (kLiveCopies - 1));
                if (any[g] & ~*p) atomicOr(p, (unsigned long long)any[g]);
            }
        }
    }
};

// What a product leaves ready for the next: the bitmaps, bounds, live columns
// and counters of F_{j+1}, last read two products ago, cleared; the vertices
// of the frontier just read and their arcs counted.
template <bool B>
__device__ __forceinline__ void quad_close(const QuadArgs &a, unsigned long long &nv, unsigned long long &na) {
    const int gtid = blockIdx.x * blockDim.x + threadIdx.x;
    const int total = gridDim.x * blockDim.x;
    close_product(a.bits, a.next_bits, a.nwords, a.nq, a.rp, a.next_ctr, nv, na);
    if constexpr (!B) return;
    const size_t count = (size_t)a.nq * a.n;
    uint32_t *p = (uint32_t *)a.lo_clear;        // the allocation is whole words
    for (size_t i = gtid; i < (count + 1) / 2; i += total) p[i] = kNone32;
    for (int i = gtid; i < a.ncg * kLiveCopies; i += total) a.live_clear[i] = 0ull;
}

template <int AM, int Q, bool COUNT, bool B, bool C>
__global__ __launch_bounds__(kBlock) MFBC_PULL_SGPRS void k_quad_pull(QuadArgs a) {
    if (!live_prev(a.prev_ctr)) {
        if constexpr (C) close_skipped(a.next_ctr);
        return;
    }
    const int wid = blockIdx.x * kWavesPerBlock + uni((int)(threadIdx.x >> 6));
    const int q = wid / a.ntasks;
    unsigned long long produced = 0, outs = 0, nv = 0, na = 0;
    if (q < a.nq) {
        QuadPull<AM, Q, COUNT, B> p(a, q);
        p.task(wid - q * a.ntasks);
        if constexpr (B) p.flush();
        produced = p.produced;
        outs = p.outs;
    }
    if constexpr (C) quad_close<B>(a, nv, na);
    flush_counts(produced, outs, nv, na, a.ctr);
}

template <int Q, bool COUNT, bool B>
__global__ __launch_bounds__(kBlock) void k_quad_merge(QuadArgs a) {
    if (!live_prev(a.prev_ctr)) {
        close_skipped(a.next_ctr);
        return;
    }
    unsigned long long nv = 0, na = 0, produced = 0, outs = 0;
    quad_close<B>(a, nv, na);
    const int wid = blockIdx.x * kWavesPerBlock + uni((int)(threadIdx.x >> 6));
    const int q = wid / a.nhubs;
    if (q < a.nq) {
        QuadPull<0, Q, COUNT, B> p(a, q);
        p.merge(wid - q * a.nhubs);
        if constexpr (B) p.flush();
        produced = p.produced;
        outs = p.outs;
    }
    flush_counts(produced, outs, nv, na, a.ctr);
}

// Nothing reached: T, bounds, bitmaps, live columns, counters.
__global__ void k_quad_init(uint32_t *t, size_t words, int32_t *hi, size_t rows, uint32_t *lo, size_t low, uint32_t *ab0,
                            uint32_t *ab1, uint32_t *ab2, uint32_t *done, size_t nab, unsigned long long *live, size_t nlive,
                            unsigned long long *ctr, int nctr, int32_t *flags) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const size_t t0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (size_t i = t0; i < words; i += stride) t[i] = kNone32;
    for (size_t i = t0; i < rows; i += stride) hi[i] = INT32_MAX;
    for (size_t i = t0; i < low; i += stride) lo[i] = kNone32;
    for (size_t i = t0; i < nab; i += stride) {
        ab0[i] = 0u;
        ab1[i] = 0u;
        ab2[i] = 0u;
        if (done) done[i] = 0u;
    }
    for (size_t i = t0; i < nlive; i += stride) live[i] = 0ull;
    for (size_t i = t0; i < (size_t)nctr; i += stride) ctr[i] = 0ull;
    if (t0 == 0) flags[0] = 0;
}

template <int Q, bool COUNT>
struct QuadSeed {
    static constexpr int kGroups = 2 * Q;
    int n, nwords;
    uint32_t *f, *t, *abits;
    uint16_t *lo;
    int32_t *off;
    const int32_t *hub;          // nullable: distance to the landmark of highest degree
    unsigned long long *live;
    uint16_t *sig;
    __device__ void row(int v, int q, int lane) const {
        Lane<Q> r;
#pragma unroll
        for (int k = 0; k < Q; k++) r.w[k] = kNone32;
        store_lane<Q>(f, (size_t)q * n + v, lane, r);
    }
    __device__ void entry(int v, int c) const {
        const int cg = c / kWave, lane = c % kWave, q = cg / kGroups, g = cg % kGroups;
        const size_t row = (size_t)q * n + v;
        const size_t i = ((row * kWave + lane) * Q + (g >> 1)) * 2 + (g & 1);
        ((uint16_t *)t)[i] = 0;
        ((uint16_t *)f)[i] = COUNT ? 1 : 0;      // weight 0, multiplicity 1 inline
        if (COUNT) sig[i] = 1;
        if (!lo) return mark(abits, q, v);
        int h = hub ? hub[v] : 0;
        if (h == kInf) h = 0;
        off[c] = h;
        const int code = kLoBias - h;
        lo[row] = (uint16_t)(code < 0 ? 0 : code);
        mark(abits, q, v);
        atomicOr(live + cg * kLiveCopies, 1ull << lane);
    }
    __device__ void mark(uint32_t *bm, int q, int v) const {
        atomicOr(bm + (size_t)q * nwords + (v >> 5), 1u << (v & 31));
    }
};

// T of one word's 128 columns (two groups) at 64 caller vertices, source by
// source.  The tile stays in 16 bits (16.6 KB of LDS, eight workgroups a CU), and
// each wave writes 64 consecutive vertices of a column at a time.  200 columns
// at n = 262,144, distances and sigma: 0.64 ms through one binary64 tile, 0.12
// + 0.31 apart.
template <int Q>
__global__ __launch_bounds__(kBlock) void k_quad_dist(const uint32_t *t, int32_t *dist, int n, int nb,
                                                      const int32_t *perm) {
    __shared__ uint32_t sh[64][65];              // [vertex][lane]: the word
    const int wd = blockIdx.y, v0 = blockIdx.x * 64;
    const int c = threadIdx.x & 63, r0 = threadIdx.x >> 6;
    uint32_t x[16];
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const int u = min(v0 + r0 + 4 * i, n - 1);
        x[i] = t[(((size_t)(wd / Q) * n + (perm ? perm[u] : u)) * kWave + c) * Q + wd % Q];
    }
#pragma unroll
    for (int i = 0; i < 16; i++) sh[r0 + 4 * i][c] = x[i];
    __syncthreads();
    const int v = v0 + c;
    if (v >= n) return;
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const int l = r0 + 4 * i;
        const uint32_t word = sh[c][l];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int s = (2 * wd + h) * kWave + l;
            const uint32_t d = half_of(word, h);
            if (s < nb) dist[(size_t)s * n + v] = d == kNone16 ? kInf : (int32_t)d;
        }
    }
}

// sigma of one word's 128 columns at 64 caller vertices, 0 where unreached: the
// tile holds the 16-bit counts, those past them are read where they are written.
template <int Q>
__global__ __launch_bounds__(kBlock) void k_quad_sigma(const uint32_t *t, const uint32_t *sig, const double *tsig,
                                                       double *sigma, int n, int nb, const int32_t *perm) {
    __shared__ uint32_t sh[64][65];              // [vertex][lane]: the word
    const int wd = blockIdx.y, v0 = blockIdx.x * 64;
    const int c = threadIdx.x & 63, r0 = threadIdx.x >> 6;
    uint32_t d[16], m[16];
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const int u = min(v0 + r0 + 4 * i, n - 1);
        const size_t at = (((size_t)(wd / Q) * n + (perm ? perm[u] : u)) * kWave + c) * Q + wd % Q;
        d[i] = t[at];
        m[i] = sig[at];
    }
#pragma unroll
    for (int i = 0; i < 16; i++)
        sh[r0 + 4 * i][c] = ((d[i] & 0xffffu) == kNone16 ? 0u : m[i] & 0xffffu) |
                            ((d[i] >> 16) == kNone16 ? 0u : m[i] & 0xffff0000u);
    __syncthreads();
    const int v = v0 + c;
    if (v >= n) return;
    const size_t dv = perm ? perm[v] : v;
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const int l = r0 + 4 * i;
        const uint32_t word = sh[c][l];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int cg = 2 * wd + h, s = cg * kWave + l;
            const uint32_t x = half_of(word, h);
            if (s < nb)
                sigma[(size_t)s * n + v] = x != kSig16Far ? (double)x : tsig[((size_t)cg * n + dv) * kWave + l];
        }
    }
}

// The batch's state after product j in the layouts of the 32-bit products, for
// product j + 1: T, path counts and, where COUNT, packed frontier tuples with
// their escaped multiplicities (FwdPull), else frontier distances (MonoPull).
// One wave per row of a wave's groups; the rows come from a copy, since the wide
// arrays lie where the 16-bit ones did.  Bound by the writes, 12 to 24 B an
// entry: 5 us for 256 columns of 3,280 vertices.  Starting over in 32 bits
// instead, ms for 256 sources on chains of cliques of 82 vertices with weights
// to 255: path counts 11.8, 9.0 so (201 products); centrality 12.2 and 10.0; with
// one weight, ties everywhere, 8.9 and 6.1 (80 products), 8.9 and 6.1.
struct WidenArgs {
    const uint32_t *t, *f;       // copies, [q][n][64][Q]
    const uint32_t *sig;
    const uint32_t *bits;        // F_j's bitmaps, [q][nwords]
    int n, nwords, nq, ncg;
    int mb16, mb;                // bits of a multiplicity, as read and as written
    int32_t *tdist;
    double *tsig, *fsig;         // fsig: F_j's, where the 16-bit form's escapes are already
    uint32_t *fw;                // F_j: [pair][n][64][2], one group [n][64]
};

template <int Q, bool COUNT>
__global__ __launch_bounds__(kBlock) void k_quad_widen(WidenArgs a) {
    const int lane = threadIdx.x & (kWave - 1);
    const size_t row = (size_t)blockIdx.x * kWavesPerBlock + (size_t)uni((int)(threadIdx.x >> 6)), n = (size_t)a.n;
    if (row >= n * (size_t)a.nq) return;
    const int q = (int)(row / n), v = (int)(row - (size_t)q * n);
    const bool act = (a.bits[(size_t)q * a.nwords + (v >> 5)] >> (v & 31)) & 1u;
    const Lane<Q> t = load_lane<Q>(a.t, row, lane);
    Lane<Q> f, s;
#pragma unroll
    for (int k = 0; k < Q; k++) f.w[k] = s.w[k] = kNone32;
    if (act) f = load_lane<Q>(a.f, row, lane);
    if constexpr (COUNT) s = load_lane<Q>(a.sig, row, lane);
    constexpr uint32_t kAbsent = COUNT ? kSent : (uint32_t)kInf;
    const uint32_t m16 = COUNT ? (1u << a.mb16) - 1u : 0u, m32 = COUNT ? (1u << a.mb) - 1u : 0u;
#pragma unroll
    for (int k = 0; k < Q; k++) {
        uint32_t w[2];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int cg = (q * Q + k) * 2 + h;
            w[h] = kAbsent;
            if (cg >= a.ncg) continue;
            const size_t i = ((size_t)cg * n + (size_t)v) * kWave + lane;
            const uint32_t d = half_of(t.w[k], h), x = half_of(f.w[k], h);
            a.tdist[i] = d == kNone16 ? kInf : (int32_t)d;
            if constexpr (COUNT) {
                const uint32_t c = half_of(s.w[k], h);
                if (d != kNone16 && c != kSig16Far) a.tsig[i] = (double)c;
                if (x != kNone16) {
                    const double m = (x & m16) != m16 ? (double)(x & m16) : a.fsig[i];
                    const uint32_t ms = m <= (double)m32 ? (uint32_t)m : 0u;
                    if (!ms) a.fsig[i] = m;
                    w[h] = ((x >> a.mb16) << a.mb) | ms;
                }
            } else if (x != kNone16) {
                w[h] = x;
            }
        }
        if (!act) continue;
        const size_t pair = (size_t)(q * Q + k);
        if (a.ncg == 1) a.fw[(size_t)v * kWave + lane] = w[0];
        else if (2 * (int)pair < a.ncg) ((uint2 *)a.fw)[(pair * n + (size_t)v) * kWave + lane] = make_uint2(w[0], w[1]);
    }
}

__global__ void k_quad_copy(const uint32_t *t, const uint32_t *f, uint32_t *t2, uint32_t *f2, size_t words) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride) {
        t2[i] = t[i];
        f2[i] = f[i];
    }
}

// F_j's bitmaps from one per Q pairs to one per pair, in place (from the last
// pair down, a pair's own plane has been read when it is written); the other two
// buffers cleared.
__global__ void k_quad_widen_bits(uint32_t *bits, uint32_t *other0, uint32_t *other1, int nwords, int npairs, int Q) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nwords) return;
    for (int p = npairs - 1; p >= 0; p--) {
        bits[(size_t)p * nwords + i] = bits[(size_t)(p / Q) * nwords + i];
        other0[(size_t)p * nwords + i] = 0u;
        other1[(size_t)p * nwords + i] = 0u;
    }
}

int grid_for(size_t work, int per, size_t cap = 0x7fffffff) {
    return (int)std::max<size_t>(1, std::min<size_t>((work + per - 1) / per, cap));
}

int bits_of(int64_t x) {
    int b = 0;
    while (x > 0) {
        b++;
        x >>= 1;
    }
    return b;
}

// Multiplicity bits of the frontier that product j reads: its candidates
// weigh at most j * maxw, and no entry may equal the all-ones one.
int quad_mb(const mfbc_graph *g, int j) { return 16 - bits_of((int64_t)j * g->maxw + 1); }

size_t quad_rows(const mfbc_graph *g, int ncg, int words) {
    return (size_t)((ncg + 2 * words - 1) / (2 * words)) * g->n;
}

QuadArgs quad_args(mfbc_graph *g, const View &vw, int ncg, int j) {
    Workspace &ws = g->ws;
    QuadArgs a{};
    const int Q = ws.quad.words, b = (j - 1) & 1;
    a.tasks = vw.plan_in.tasks;
    a.hubs = vw.plan_in.hubs;
    a.ntasks = vw.plan_in.ntasks;
    a.nhubs = vw.plan_in.nhubs;
    a.nslots = vw.plan_in.nslots;
    a.ncg = ncg;
    a.n = g->n;
    a.nwords = (g->n + 31) / 32;
    a.nq = (ncg + 2 * Q - 1) / (2 * Q);
    a.rp = vw.in.rp;
    a.arcs.col = vw.in.col;
    a.arcs.w = vw.in.w;
    a.arcs.pk = vw.in.pk;
    a.arcs.cb = vw.in.cb;
    a.arcs.cmask = vw.in.cb >= 32 ? 0xffffffffu : ((1u << vw.in.cb) - 1u);
    a.owner = vw.plan_in.owner;
    a.f = (const uint32_t *)ws.fdist[b];
    a.f_n = (uint32_t *)ws.fdist[b ^ 1];
    a.t = (uint32_t *)ws.tdist;
    const QuadBounds &qb = ws.quad;
    a.lo = qb.lo[(j - 1) % 3];
    a.lo_n = qb.lo[j % 3];
    a.lo_clear = qb.lo[(j + 1) % 3];
    a.hi = qb.hi;
    a.off = qb.off;
    const size_t nlive = (size_t)ncg * kLiveCopies;
    a.live = qb.live + (size_t)((j - 1) % 3) * nlive;
    a.live_n = qb.live + (size_t)(j % 3) * nlive;
    a.live_clear = qb.live + (size_t)((j + 1) % 3) * nlive;
    // the backward half's lane masks, not in use yet, hold the bitmap
    a.done = !ws.quad.hi && !vw.in.w && !vw.in.pk ? (uint32_t *)ws.fbits[0] : nullptr;
    a.src = ws.src;
    a.bits = ws.abits[(j - 1) % 3];
    a.bits_n = ws.abits[j % 3];
    a.next_bits = ws.abits[(j + 1) % 3];
    a.pd = ws.pd;
    a.pm = ws.pm;
    a.ctr = ws.counters + (size_t)(j % kCounterRing) * 4 * kCounterSlots;
    a.prev_ctr = j > 1 ? ws.counters + (size_t)((j - 1) % kCounterRing) * 4 * kCounterSlots : nullptr;
    a.next_ctr = ws.counters + (size_t)((j + 1) % kCounterRing) * 4 * kCounterSlots;
    a.mb = quad_mb(g, j);
    a.mbn = quad_mb(g, j + 1);
    a.sig = ws.tau2;
    a.tsig = ws.tsig;
    a.fsig = ws.fsig[b];
    a.fsig_n = ws.fsig[b ^ 1];
    a.flags = ws.flags;
    return a;
}

template <int Q, bool COUNT, bool B>
void quad_init(mfbc_graph *g, const View &vw, int ncg, int nb, const int32_t *d_sources, hipStream_t s) {
    const QuadArgs a = quad_args(g, vw, ncg, 1);
    Workspace &ws = g->ws;
    const size_t rows = (size_t)a.nq * g->n, words = rows * kWave * Q;
    hipLaunchKernelGGL(k_quad_init, dim3(grid_for(words, 1024, 16384)), dim3(256), 0, s, a.t, words, a.hi,
                       B ? rows : 0, (uint32_t *)ws.quad.lo[0], B ? 3 * ws.quad.lo_words : 0, ws.abits[0], ws.abits[1],
                       ws.abits[2], a.done, (size_t)a.nq * a.nwords, ws.quad.live, B ? (size_t)3 * ncg * kLiveCopies : 0,
                       ws.counters, (int)kRingWords, ws.flags);
    const QuadSeed<Q, COUNT> seed{g->n,    a.nwords,  (uint32_t *)ws.fdist[0], a.t, ws.abits[0], ws.quad.lo[0],
                                  ws.quad.off, g->hub_dist, ws.quad.live, (uint16_t *)a.sig};
    launch_seed(g, seed, ncg, nb, d_sources, s);
}

template <int AM, int Q, bool COUNT, bool B>
void quad_pull(const QuadArgs &a, int grid, hipStream_t s) {
    if (a.nhubs) hipLaunchKernelGGL((k_quad_pull<AM, Q, COUNT, B, false>), dim3(grid), dim3(kBlock), 0, s, a);
    else hipLaunchKernelGGL((k_quad_pull<AM, Q, COUNT, B, true>), dim3(grid), dim3(kBlock), 0, s, a);
}

template <int Q, bool COUNT, bool B>
void quad_product(mfbc_graph *g, const View &vw, int ncg, int j, hipStream_t s, hipEvent_t *ev) {
    const QuadArgs a = quad_args(g, vw, ncg, j);
    if (ev) (void)hipEventRecord(ev[0], s);
    const int grid = grid_for((size_t)a.ntasks * a.nq, kWavesPerBlock);
    const Csr &c = vw.in;
    if (c.pk) quad_pull<1, Q, COUNT, B>(a, grid, s);
    else if (c.w) quad_pull<2, Q, COUNT, B>(a, grid, s);
    else quad_pull<0, Q, COUNT, B>(a, grid, s);
    if (ev) (void)hipEventRecord(ev[1], s);
    if (a.nhubs) {
        const int mgrid = std::max(grid_for((size_t)a.nhubs * a.nq, kWavesPerBlock),
                                   grid_for((size_t)a.nwords, kBlock, 1024));
        hipLaunchKernelGGL((k_quad_merge<Q, COUNT, B>), dim3(mgrid), dim3(kBlock), 0, s, a);
    }
    if (ev && ev[2]) (void)hipEventRecord(ev[2], s);
}

template <int Q, bool COUNT, bool B>
void quad_widen(mfbc_graph *g, const View &vw, int ncg, int j, hipStream_t s) {
    Workspace &ws = g->ws;
    const QuadArgs a = quad_args(g, vw, ncg, j);
    const size_t rows = (size_t)a.nq * g->n, words = rows * kWave * Q;
    // the multiplicities of F_{j-1} are done with: room for both copies
    uint32_t *t2 = (uint32_t *)ws.fsig[(j & 1) ^ 1], *f2 = t2 + words;
    hipLaunchKernelGGL(k_quad_copy, dim3(grid_for(words, 1024, 16384)), dim3(256), 0, s, (const uint32_t *)a.t,
                       (const uint32_t *)a.f_n, t2, f2, words);
    WidenArgs w{};
    w.t = t2;
    w.f = f2;
    w.sig = a.sig;
    w.bits = a.bits_n;
    w.n = a.n;
    w.nwords = a.nwords;
    w.nq = a.nq;
    w.ncg = ncg;
    w.mb16 = a.mbn;
    w.mb = g->mb;
    w.tdist = ws.tdist;
    w.tsig = ws.tsig;
    w.fsig = ws.fsig[j & 1];
    w.fw = (uint32_t *)ws.fdist[j & 1];
    hipLaunchKernelGGL((k_quad_widen<Q, COUNT>), dim3(grid_for(rows, kWavesPerBlock)), dim3(kBlock), 0, s, w);
    hipLaunchKernelGGL(k_quad_widen_bits, dim3(grid_for(a.nwords, 256)), dim3(256), 0, s, a.bits_n,
                       ws.abits[(j + 1) % 3], ws.abits[(j + 2) % 3], a.nwords, (ncg + 1) / 2, Q);
}

template <int Q, bool COUNT>
void quad_rows_out(mfbc_graph *g, int ncg, int nb, int32_t *dist, double *sigma, hipStream_t s) {
    const uint32_t *t = (const uint32_t *)g->ws.tdist;
    const int32_t *perm = g->perm;
    hipLaunchKernelGGL(k_quad_dist<Q>, dim3((g->n + 63) / 64, (ncg + 1) / 2), dim3(kBlock), 0, s, t, dist, g->n, nb,
                       perm);
    if constexpr (COUNT)
        hipLaunchKernelGGL(k_quad_sigma<Q>, dim3((g->n + 63) / 64, (ncg + 1) / 2), dim3(kBlock), 0, s, t,
                           (const uint32_t *)g->ws.tau2, (const double *)g->ws.tsig, sigma, g->n, nb, perm);
}

}  // namespace

// Products whose entries fit 16 bits, in whole windows; 0 where so few do
// that most of a call would run in 32 bits all the same.  Distances need j *
// maxw < 65535, multiplicities two bits besides: weights up to 255 fit 56
// products with multiplicities (most graphs take 10 to 25), 256 without.  A
// graph of short rows (grids, paths) may take any number of products and has
// to fit whole (no shortest path has more arcs than vertices).  Centrality of
// 256 sources, ms in 32 bits throughout / in 16 as far as they go: a grid of 30
// by 30 with weights to 255, 62 products, 1.76 / 1.76; of 100 by 100, 211
// products, 11.6 / 11.7; uniform of degree 10, n = 10,000, 900 sources 5.1 /
// 4.9, n = 100,000 8.1 / 6.1.
int quad_products(const mfbc_graph *g, bool count) {
    constexpr int kLeast = 40;
    const int64_t most = count ? ((int64_t)1 << 14) - 1 : 65535;
    const int64_t j = (most - 1) / g->maxw - (count ? 1 : 0);     // product j writes for product j + 1
    const int64_t fit = j / kWindow * kWindow;
    return fit < kLeast || (g->sparse && g->n > fit) ? 0 : (int)std::min<int64_t>(fit, 1 << 20);
}

size_t quad_bound_bytes(const mfbc_graph *g, int ncg, int words, QuadBounds *qb, char *base) {
    const size_t rows = quad_rows(g, ncg, words);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *p = base ? base + off : nullptr;
        off = (off + bytes + 255) & ~(size_t)255;
        return p;
    };
    QuadBounds b;
    b.words = words;
    b.lo_words = (rows + 1) / 2;
    uint16_t *lo = (uint16_t *)take(3 * b.lo_words * 4);
    for (int i = 0; i < 3; i++) b.lo[i] = lo ? lo + (size_t)i * 2 * b.lo_words : nullptr;
    b.hi = (int32_t *)take(rows * 4);
    b.off = (int32_t *)take((size_t)ncg * kWave * 4);
    b.live = (unsigned long long *)take((size_t)3 * ncg * kLiveCopies * 8);
    if (qb) *qb = b;
    return off;
}

// The forms in use: with bounds, one or two words a lane, with multiplicities
// or without; and one word with multiplicities without bounds (a core).
#define MFBC_QUAD(fn, ...)                                              \
    do {                                                                \
        if (!g->ws.quad.hi) fn<1, true, false>(__VA_ARGS__);            \
        else if (g->ws.quad.words == 1 && count) fn<1, true, true>(__VA_ARGS__); \
        else if (g->ws.quad.words == 1) fn<1, false, true>(__VA_ARGS__);         \
        else if (count) fn<2, true, true>(__VA_ARGS__);                 \
        else fn<2, false, true>(__VA_ARGS__);                           \
    } while (0)

void launch_quad_init(mfbc_graph *g, const View &vw, bool count, int ncg, int nb, const int32_t *d_sources,
                      hipStream_t s) {
    MFBC_QUAD(quad_init, g, vw, ncg, nb, d_sources, s);
}
void launch_quad_product(mfbc_graph *g, const View &vw, bool count, int ncg, int j, hipStream_t s,
                         hipEvent_t *ev) {
    MFBC_QUAD(quad_product, g, vw, ncg, j, s, ev);
}
void launch_quad_widen(mfbc_graph *g, const View &vw, bool count, int ncg, int j, hipStream_t s) {
    MFBC_QUAD(quad_widen, g, vw, ncg, j, s);
}
void launch_quad_rows(mfbc_graph *g, bool count, int ncg, int nb, int32_t *dist, double *sigma, hipStream_t s) {
    if (g->ws.quad.words == 1 && count) quad_rows_out<1, true>(g, ncg, nb, dist, sigma, s);
    else if (g->ws.quad.words == 1) quad_rows_out<1, false>(g, ncg, nb, dist, sigma, s);
    else if (count) quad_rows_out<2, true>(g, ncg, nb, dist, sigma, s);
    else quad_rows_out<2, false>(g, ncg, nb, dist, sigma, s);
}

}  // namespace mfbc
