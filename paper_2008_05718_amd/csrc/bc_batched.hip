// bc_batched.hip -- batched Brandes engine: up to 64 sources traversed
// together, one wavefront lane per source.
//
// The paper's forward phase exploits that BC needs a traversal from many
// sources (Section "Introduction" and "Comparison with Totem": one-time work
// amortised over many sources).  Here that multi-source property becomes the
// batching axis: the frontier of a level is one list of vertices, each with a
// 64-bit lane mask (bit k = the vertex is on this level for source k), so a
// vertex's adjacency is read once per level for all sources that reach it
// there.  Per-source state lives in vertex-major slabs [n][64] (sigma, then
// delta; and c = (1 + delta) / sigma), so the 64 lanes of a wavefront touch
// one contiguous 512-byte row.
//
// Per level l (Algorithm "Betweenness Centrality Algorithm", forward loop):
//   PH_FWD  discover: visited/next words, push (packed group or wavefront per
//           frontier vertex, 64-bit atomicOr) or pull (thread per unvisited
//           vertex, four arcs at a time, early exit once every needed lane is
//           found).
//   PH_SIG  sigma_k(w) = sum over neighbours u of w on level l in lane k of
//           sigma_k(u), in CSR order, one wavefront per new vertex.  uint64
//           with the carry kept (exact overflow test); scaled FP64 in mode 1.
// Backward, per level l = L-1 .. 1 (same figure, backward loop; Eq. 2):
//   PH_BWD  delta_k(v) = sigma_k(v) * sum over w on level l+1 of c_k(w).
//   PH_BC   BC[v] += delta_k(v) for k = 0 .. 63 in order (source-list
//           order), then the visited words are cleared.
// Frontier words carry a level tag so stale entries never need clearing.
//
// Load balance: sums and pushes work on groups of level entries of about equal
// cost; in a group the arcs of vertices of degree <= kPack are packed into
// 64-arc chunks, a vertex of up to a segment of arcs has the wavefront to itself,
// and a heavier one is split into segments, one wavefront each (pull: one
// thread per vertex up to kLightDeg).  Segment partial sums are combined in
// segment order by the last segment to finish, so every sum has an order fixed
// by the vertex and the results are bitwise reproducible.
#include "bc_common.h"

#ifndef BC_UNROLL
#define BC_UNROLL 16
#endif
namespace bcx {
constexpr int kUnroll = BC_UNROLL;  // matched neighbours whose rows are loaded together
}
#include "bc_rows.h"

namespace bcx {

// ------------------------------------------------------------------ pieces

// Where a discover step appends the next level.
template <class To>
struct Append {
    const To &to;
    Stage &st;
    int n;  // staged entries (wavefront-uniform)
};
template <class To>
__device__ __forceinline__ void append(Append<To> &ap, bool pred, int w) {
    stage_push(pred, w, ap.st, ap.n, ap.to);
}

// Push over the arc of each thread (far end w with visited/next words x, lanes
// f of the arc's tail): vertices reached for the first time on the next level
// are appended.
template <class To>
__device__ __forceinline__ void push_arc(const BatchArgs &a, Append<To> &ap, int w, unsigned long long f, VisNext x) {
    const unsigned long long add = f & ~x.vis & ~x.nxt;
    bool newly = false;
    if (add) newly = atomicOr(&a.vn[w].nxt, add) == 0ull;
    append(ap, newly, w);
}

// Push from one frontier vertex (lanes f) over arcs [a0, a1) (uniform), 64 at a
// time; the next chunk's columns and words are requested first.
template <class To>
__device__ __forceinline__ void push_arcs(const BatchArgs &a, Append<To> &ap, unsigned long long f, int a0, int a1,
                                          const int32_t *__restrict__ col) {
    if (a0 >= a1) return;
    const int lane = lane_id(), n = a1 - a0;
    col += a0;
    int w = col[min(lane, n - 1)], wn = col[min(kWave + lane, n - 1)];
    VisNext x = a.vn[w];
    for (int i = 0; i < n; i += kWave) {
        const int wc = w;
        const VisNext xc = x;
        if (i + kWave < n) {
            w = wn;
            x = a.vn[w];
            wn = col[min(i + 2 * kWave + lane, n - 1)];
        }
        push_arc(a, ap, wc, i + lane < n ? f : 0ull, xc);
    }
}

// Push from a group of frontier entries: light ones packed like the sums'
// groups, medium ones one at a time.  Returns (lane 0) the arcs followed.
template <class To>
__device__ __forceinline__ unsigned push_group(const BatchArgs &a, Append<To> &ap, Packing &pk, int qb, int i0, int i1,
                                               unsigned long long act, const int32_t *__restrict__ rp,
                                               const int32_t *__restrict__ col) {
    const int lane = lane_id();
    const bool valid = i0 + lane < i1;
    const int p = qb + i0 + lane;
    const int u = valid ? a.lq_vtx[p] : 0;
    const unsigned long long f = valid ? (a.lq_mask[p] & act) : 0ull;
    const int e0 = f ? rp[u] : 0, od = f ? rp[u + 1] - e0 : 0;  // out-arcs to push over
    const int deg = f ? class_deg(a.g, u, od) : 0;
    const bool light = f && deg <= kPack, medium = f && deg > kPack && deg <= seg_arcs(a.g);
    int off;
    const int total = pack_entries(pk, light ? od : 0,
                                   make_uint4((unsigned)e0, (unsigned)f, (unsigned)(f >> 32), 0u),
                                   make_uint4(0u, 0u, 0u, 0u), off);
    unsigned arcs = (unsigned)total;
    if (total) {
        int before = 0;
        uint4 r = pk.rec[packed_rank(pk, 0, before)], rn = r;
        int w = col[(int)r.x + min(lane, total - 1)], wn = w;
        VisNext x = a.vn[w];
        if (kWave < total) {
            rn = pk.rec[packed_rank(pk, 1, before)];
            wn = col[(int)rn.x + min(kWave + lane, total - 1)];
        }
        for (int base = 0; base < total; base += kWave) {
            const int wc = w;
            const VisNext xc = x;
            const unsigned long long fc = base + lane < total ? (((unsigned long long)r.z << 32) | r.y) : 0ull;
            if (base + kWave < total) {
                w = wn;
                r = rn;
                x = a.vn[w];
                if (base + 2 * kWave < total) {
                    rn = pk.rec[packed_rank(pk, base / kWave + 2, before)];
                    wn = col[(int)rn.x + min(base + 2 * kWave + lane, total - 1)];
                }
            }
            push_arc(a, ap, wc, fc, xc);
        }
    }
    for (unsigned long long mm = __ballot(medium); mm; mm &= mm - 1) {
        const int j = __ffsll(mm) - 1;
        const int a0 = __builtin_amdgcn_readlane(e0, j), n = __builtin_amdgcn_readlane(od, j);
        push_arcs(a, ap, readlane_u64(f, j), a0, a0 + n, col);
        arcs += (unsigned)n;
    }
    wave_lds_fence();  // the next group reuses the packing
    return lane == 0 ? arcs : 0u;
}

// New vertex w (queue position p, visited/next words vis/m, degree deg)
// joins the level-(l+1) frontier; called by one thread per entry.
__device__ __forceinline__ void sig_publish(const BatchArgs &a, Tagged *fw_nxt, uint32_t T1, int p, int w,
                                            unsigned long long vis, unsigned long long m, int deg,
                                            unsigned long long lmask, SigCounters &sc) {
    VisNext y;
    y.vis = vis | m;
    y.nxt = 0ull;
    a.vn[w] = y;
    Tagged tg;
    tg.mask = m;
    tg.tag = T1;
    fw_nxt[w] = tg;
    a.lq_mask[p] = m;
    sc.edges += (unsigned)deg;
    sc.act |= m;
    sc.lent += (unsigned)__popcll(m);
    if ((y.vis & lmask) == lmask) {
        sc.full_n += 1;
        sc.full_m += (unsigned)deg;
    }
}

// LDS scratch of one wavefront, one use at a time.
union WaveScratch {
    struct {
        Packing pk;             // sums and push: a group's packed entries
        Stage st;               // discover: staged queue entries
    } w;
    double tile[kWave * 8];     // score accumulation: 64 rows x 8 lanes
};

// Path counts for the entries [i0, i1) of level l+1 (one group):
// entries of degree <= kPack have their adjacencies packed into dense 64-arc
// chunks; entries of up to a segment follow one at a time; heavier ones run as
// segments elsewhere.  Every entry's sum keeps CSR order.
//
// What bounds it: on R-MAT 22 the bytes fetched beyond the L2 (5.8 TB/s: a
// matched row has 16 of 64 lanes in use but touches 2.8 of its four 128-byte
// lines), on smaller graphs the latency of the chain entry -> row offsets ->
// column -> frontier word -> row and the instructions per match.  Rows as
// scalar buffers, records by bit counting, one load per frontier word and
// loads a chunk ahead, against vector addresses, searches across lanes and
// tag-then-mask loads: path-count and backward device time on R-MAT 18 (2048
// sources, summed over 8 replicas) 90 + 95 -> 70 + 85 ms, R-MAT 22 (1024
// sources, 4 replicas) 342 + 439 -> 327 + 385 ms; ER(2000), all sources, in the
// block engine 7.1 -> 5.0 ms.  Matches at a time, 4 / 8 / 16 / 24 / 32: R-MAT 18,
// 2048 sources, 35.3 / 31.6 / 30.2 / 31.2 / 33.3 ms a run, R-MAT 22, 1024 sources,
// 279.7 / 264.6 / 261.0 / 265.8 / 278.6 (where a register or two more spill, the
// gain is lost).
template <int MODE>
__device__ __forceinline__ void sig_group(const BatchArgs &a, const Tagged *fw_cur, Tagged *fw_nxt, uint32_t T, int qs,
                                          int i0, int i1, int sh, unsigned long long lmask, SigCounters &sc, int l,
                                          int *s_emax, int *s_emin, float il, Packing &pk) {
    constexpr int OP = MODE ? OP_F64 : OP_U64;
    // predecessors: the in-arcs (the adjacency itself for undirected graphs)
    const int32_t *__restrict__ rp = a.g.in_row_ptr;
    const int32_t *__restrict__ col = a.g.in_col;
    const int lane = lane_id();
    const int i = i0 + lane;
    const bool valid = i < i1;
    const int p = qs + i;
    const int w = valid ? a.lq_vtx[p] : 0;
    const int e0 = valid ? rp[w] : 0;
    const int na = valid ? rp[w + 1] - e0 : 0;  // arcs to scan
    const int od = (valid && a.g.directed) ? a.g.row_ptr[w + 1] - a.g.row_ptr[w] : na;  // out-degree
    const int deg = a.g.directed ? (valid ? max(na, od) : 0) : na;  // class degree
    const bool light = valid && deg <= kPack;
    const bool medium = valid && deg > kPack && deg <= seg_arcs(a.g);
    unsigned long long vis = 0, nxt = 0;
    if (light || medium) {
        const VisNext x = a.vn[w];
        vis = x.vis;
        nxt = x.nxt;
    }
    const unsigned long long ra = row_addr(a.sigma, w);
    const unsigned long long limit = a.sigma_limit;
    unsigned long long ovf = 0;  // lanes whose counts overflowed (wavefront-uniform)
    // few sources per light entry: one thread per (entry, source) pair
    const int n_items = (int)wave_sum_u32(light ? (unsigned)__popcll(nxt) : 0u);
    const int n_light = __popcll(__ballot(light));
    int off;
    if (n_light > 0 && (float)n_items <= il * (float)n_light) {
        pack_entries(pk, light ? __popcll(nxt) : 0,
                     make_uint4(0u, (unsigned)nxt, (unsigned)(nxt >> 32), (unsigned)w),
                     make_uint4((unsigned)e0, (unsigned)na, 0u, 0u), off);
        int before = 0;
        for (int c = 0; c * kWave < n_items; ++c) {
            const int rank = packed_rank(pk, c, before);
            const int it = c * kWave + lane;
            if (it < n_items) {
                const uint4 r = pk.rec[rank], r2 = pk.rec2[rank];
                const int k = nth_set_bit(((unsigned long long)r.z << 32) | r.y, it - (int)r2.z);
                const int shk = MODE ? a.shift[(size_t)l * kLanes + k] : 0;
                RowSum<OP> s;
                const unsigned matched = item_arcs(fw_cur, T, k, (int)r2.x, (int)(r2.x + r2.y), col, a.sigma,
                                                   [&](unsigned long long v) { s.add(v, shk); });
                sc.ac.larcs += matched;
                sc.ac.pairs += matched;
                sc.ac.arcs += r2.y;
                a.sigma[(size_t)r.w * kLanes + k] = MODE ? as_u64(s.d) : s.lo;
                if (MODE == 0) {
                    if (s.hi != 0u || s.lo > a.sigma_limit) sc.ovf |= 1ull << k;
                } else if (s.d > 0.0) {
                    int ex;
                    frexp(s.d, &ex);
                    atomicMax(&s_emax[k], ex);
                    atomicMin(&s_emin[k], ex);
                }
            }
        }
    } else if (n_light > 0) {
        const int total = pack_entries(pk, light ? na : 0,
                                       make_uint4((unsigned)e0, (unsigned)nxt, (unsigned)(nxt >> 32), (unsigned)lane),
                                       make_uint4(0u, 0u, 0u, 0u), off);
        RowSum<OP> acc;
        int cur;
        // every entry was discovered through an arc from level l in each of
        // its lanes, so every entry has a match
        auto fin = [&](int e, const RowSum<OP> &s) {
            sig_store<OP>(s, readlane_u64(nxt, e), readlane_u64(ra, e), limit, ovf, sc);
        };
        row_packed<OP>(pk, total, TagLanes{fw_cur, T}, sh, col, a.sigma, acc, cur, sc.ac, fin);
        if (cur >= 0) fin(cur, acc);
    }
    // medium-degree entries: one wavefront-wide scan each
    for (unsigned long long mm = __ballot(medium); mm; mm &= mm - 1) {
        const int j = __ffsll(mm) - 1;
        const int a0 = __builtin_amdgcn_readlane(e0, j), dj = __builtin_amdgcn_readlane(na, j);
        const unsigned long long mj = readlane_u64(nxt, j);
        RowSum<OP> acc;
        row_arcs<OP>(TagLanes{fw_cur, T}, mj, a0, a0 + dj, sh, col, a.sigma, acc, sc.ac);
        sig_store<OP>(acc, mj, readlane_u64(ra, j), limit, ovf, sc);
    }
    sc.ovf |= ovf;
    if (light || medium) sig_publish(a, fw_nxt, T + 1u, p, w, vis, nxt, od, lmask, sc);
    wave_lds_fence();  // the next group reuses the packing
}

// Dependencies for the entries [i0, i1) of level l (one group), packed like
// sig_group.  A complete sum is parked in the entry's delta row; at the end of
// the group the rows are taken up again four entries at a time, together with
// their path counts (one entry at a time, that load stood at the end of the
// chain of every entry).
template <int MODE>
__device__ __forceinline__ void bwd_group(const BatchArgs &a, const Tagged *fb_nxt, Tagged *fb_cur, uint32_t TB,
                                          int qb, int i0, int i1, unsigned long long dead, int sh, int shn,
                                          ArcCounters &ac, int l, bool has_next, float il, Packing &pk) {
    const int32_t *__restrict__ rp = a.g.row_ptr;
    const int32_t *__restrict__ col = a.g.col;
    const int lane = lane_id();
    const int i = i0 + lane;
    const bool valid = i < i1;
    const int p = qb + i;
    const int v = valid ? a.lq_vtx[p] : 0;
    const int e0 = valid ? rp[v] : 0;
    const int na = valid ? rp[v + 1] - e0 : 0;  // successors: the out-arcs
    const int deg = valid ? class_deg(a.g, v, na) : 0;
    const bool light = valid && deg <= kPack;
    const bool medium = valid && deg > kPack && deg <= seg_arcs(a.g);
    const unsigned long long Mf = (light || medium) ? a.lq_mask[p] : 0ull;
    const unsigned long long M = Mf & ~dead;
    unsigned long long todo = 0, parked = 0;  // entries to finish below; those with a sum in their delta row
    // few sources per light entry: one thread per (entry, source) pair
    const int n_items = (int)wave_sum_u32(light ? (unsigned)__popcll(M) : 0u);
    const int n_light = __popcll(__ballot(light));
    int off;
    if (n_light > 0 && (float)n_items <= il * (float)n_light) {
        pack_entries(pk, light ? __popcll(M) : 0, make_uint4(0u, (unsigned)M, (unsigned)(M >> 32), (unsigned)v),
                     make_uint4((unsigned)e0, (unsigned)na, 0u, 0u), off);
        int before = 0;
        for (int c = 0; c * kWave < n_items; ++c) {
            const int rank = packed_rank(pk, c, before);
            const int it = c * kWave + lane;
            if (it < n_items) {
                const uint4 r = pk.rec[rank], r2 = pk.rec2[rank];
                const int k = nth_set_bit(((unsigned long long)r.z << 32) | r.y, it - (int)r2.z);
                const size_t at = (size_t)r.w * kLanes + k;
                const unsigned long long raw = a.sigma[at];
                RowSum<OP_C> s;
                const unsigned matched =
                    item_arcs(fb_nxt, TB + 1u, k, (int)r2.x, (int)(r2.x + r2.y), col,
                              (const unsigned long long *)a.chat, [&](unsigned long long x) { s.add(x, 0); });
                ac.larcs += matched;
                ac.pairs += matched;
                ac.arcs += r2.y;
                const int shk = MODE ? a.shift[(size_t)l * kLanes + k] : 0;
                const int shnk = (MODE && has_next) ? a.shift[(size_t)(l + 1) * kLanes + k] : 0;
                double delta, cc;
                bwd_values<MODE>(raw, s.d, shk, shnk, delta, cc);
                a.chat[at] = cc;
                a.delta[at] = delta;
            }
        }
    } else if (n_light > 0) {
        const int total = pack_entries(pk, (light && M) ? na : 0,
                                       make_uint4((unsigned)e0, (unsigned)M, (unsigned)(M >> 32), (unsigned)lane),
                                       make_uint4(0u, 0u, 0u, 0u), off);
        RowSum<OP_C> acc;
        int cur;
        auto fin = [&](int e, const RowSum<OP_C> &s) {
            row_store(row_addr(a.delta, __builtin_amdgcn_readlane(v, e)), row_slot(readlane_u64(M, e)), as_u64(s.d));
            parked |= 1ull << e;
        };
        row_packed<OP_C>(pk, total, TagLanes{fb_nxt, TB + 1u}, 0, col, a.chat, acc, cur, ac, fin);
        if (cur >= 0) fin(cur, acc);
        todo = __ballot(light && M != 0ull);
    }
    for (unsigned long long mm = __ballot(medium && M != 0ull); mm; mm &= mm - 1) {
        const int j = __ffsll(mm) - 1;
        const int a0 = __builtin_amdgcn_readlane(e0, j), dj = __builtin_amdgcn_readlane(na, j);
        const unsigned long long mj = readlane_u64(M, j);
        RowSum<OP_C> acc;
        row_arcs<OP_C>(TagLanes{fb_nxt, TB + 1u}, mj, a0, a0 + dj, 0, col, a.chat, acc, ac);
        row_store(row_addr(a.delta, __builtin_amdgcn_readlane(v, j)), row_slot(mj), as_u64(acc.d));
        parked |= 1ull << j;
        todo |= 1ull << j;
    }
    bwd_finish<MODE>(todo, parked, M, v, a.sigma, a.chat, a.delta, sh, shn);
    if (light || medium) {
        Tagged tg;
        tg.mask = Mf;
        tg.tag = TB;
        fb_cur[v] = tg;
    }
    wave_lds_fence();  // the next group reuses the packing
}

// Lanes of `need` found on the level with tag T among the far ends of arcs
// [a0, a1) (uniform), 64 at a time until every needed lane is found.
__device__ __forceinline__ unsigned long long pull_arcs(const Tagged *fw, uint32_t T, unsigned long long need, int a0,
                                                        int a1, const int32_t *__restrict__ col, int &scanned) {
    unsigned long long got = 0;
    if (!need || a0 >= a1) return 0ull;
    const int lane = lane_id(), n = a1 - a0;
    col += a0;
    int u = col[min(lane, n - 1)];
    for (int i = 0; i < n && got != need; i += kWave) {
        const unsigned long long f = tagged_lanes(fw, u, T, need);  // (the last arc again beyond the end)
        if (i + kWave < n) u = col[min(i + kWave + lane, n - 1)];
        got |= wave_or_u64(f);
        scanned += min(kWave, n - i);
    }
    return got;
}

// The variant of the next level and the summation options chosen with it
// (lbo, see choose_variant); when collecting timings, every level starts
// with variant 0 and its normalised features are kept for the samples.
__device__ __forceinline__ void set_level_variant(const BatchArgs &a, Head *c, int v, int lbo, const LevelFeatures &f,
                                                  float n, float nnz) {
    if (f.level < a.max_levels + 2) a.lbsel[f.level] = lbo;
    if (c->collect) {
        float x[kMlpIn];
        mlp_inputs(f, n, nnz, x);
        for (int i = 0; i < kMlpIn; ++i) c->feat[i] = x[i];
        if (a.col_F && f.level < a.max_levels + 2)
            for (int i = 0; i < kMlpIn; ++i) a.col_F[(size_t)f.level * kMlpIn + i] = x[i];
        c->cvar = 0;
        c->variant = 0;
    } else {
        c->variant = v;
    }
}

// Where a machine counts its steps on level l.
__device__ __forceinline__ LevelRec &level_of(const Ctl *, const BatchArgs &a, int l) { return level_rec(a.lvl, l); }
__device__ __forceinline__ LevelRec &level_of(SoloCtl *c, const BatchArgs &a, int l) {
    return l < kSoloLevels ? c->lvl[l] : level_rec(a.lvl, l);
}

template <int MODE, class C>
__device__ __forceinline__ void batch_begin(const BatchArgs &a, C *gc, Head *c, int64_t b, float *lds, LevelFeatures *sf,
                                            int *s_lsrc, int *s_cnt, unsigned long long *s_tmp, int *s_lead) {
    const int t = threadIdx.x;
    const int64_t start = a.batch_start[b], end = a.batch_start[b + 1];
    const int lanes = (int)(end - start);
    // Tags of the previous batch end at epoch_b + n_levels; start above them.
    const uint32_t epoch = c->epoch_b + (uint32_t)c->n_levels + 1u;
    __syncthreads();
    if (t == 0) *s_cnt = 0;
    if (t < kLanes) {
        const int s = t < lanes ? a.srcs[start + t] : -1;
        s_lsrc[t] = s;
        a.lane_src[t] = s;
        c->lane_E[t] = 0;
        c->lane_emax[t] = INT_MIN;
    }
    __syncthreads();
    // lanes with the same source share one level-0 entry, led by its lowest lane
    unsigned long long m = 0;
    int lead = t;
    if (t < lanes) {
        const int s = s_lsrc[t];
        for (int k = lanes - 1; k >= 0; --k) {
            if (s_lsrc[k] == s) {
                m |= 1ull << k;
                lead = k;
            }
        }
        s_lead[t] = lead;
    }
    __syncthreads();
    if (t < lanes) {
        const int s = s_lsrc[t];
        a.sigma[(size_t)s * kLanes + t] = MODE ? as_u64(1.0) : 1ull;
        if (lead == t) {
            const int j = atomicAdd(s_cnt, 1);
            a.lq_vtx[j] = s;
            a.lq_mask[j] = m;
            a.vn[s].vis = m;
            Tagged tg;
            tg.mask = m;
            tg.tag = epoch;
            a.fw0[s] = tg;
            const int od = a.g.row_ptr[s + 1] - a.g.row_ptr[s];
            s_tmp[j] = (unsigned long long)(unsigned)od | ((unsigned long long)(unsigned)class_deg(a.g, s, od) << 32);
        }
    }
    if (MODE && t < kLanes) a.shift[t] = 0;
    __syncthreads();
    if (t == 0) {
        const int cnt = *s_cnt;
        unsigned long long mf = 0;
        uint32_t cost = 0;
        int nh = 0, segs = 0;
        for (int j = 0; j < cnt; ++j) {
            const int deg = (int)(uint32_t)s_tmp[j], cdeg = (int)(s_tmp[j] >> 32);
            mf += (unsigned long long)deg;
            const uint32_t ce = entry_cost(cdeg, a.g.seg_log);
            for (uint32_t k = cost / kBudget + 1; k <= (cost + ce) / kBudget; ++k) a.gstart[k] = (uint32_t)j + 1u;
            cost += ce;
            if (cdeg > seg_arcs(a.g)) {  // heavy source: level-0 segments for the push
                a.hq.pos[nh] = j;
                a.hq.seg[nh] = segs;
                a.hq.cnt[nh] = 0;
                segs += n_segments(a.g, cdeg);
                ++nh;
            }
        }
        a.hq.off[0] = 0;
        a.hq.off[1] = nh;
        a.hq.nseg[0] = segs;
        const uint32_t ng = (cost - 1u) / (uint32_t)kBudget + 1u;  // groups of level 0
        a.gstart[0] = 0u;
        a.gstart[ng] = (uint32_t)cnt;
        a.gbase[0] = 0u;
        a.gbase[1] = ng + 1u;
        c->epoch = epoch;
        c->pos = b;
        c->lanes = lanes;
        c->lane_mask = lanes >= 64 ? ~0ull : ((1ull << lanes) - 1ull);
        c->active = c->lane_mask;
        c->dead = 0;
        c->range_lo = a.batch_lo[b];
        c->range_hi = a.batch_hi[b];
        c->range_arcs = (unsigned long long)(a.g.row_ptr[c->range_hi] - a.g.row_ptr[c->range_lo]);
        c->range_nodeg = (unsigned long long)(c->range_hi - c->range_lo);
        c->full_n = 0;
        c->full_m = 0;
        c->level = 0;
        c->n_levels = 0;
        a.level_off[0] = 0;
        a.level_off[1] = cnt;
        c->prev_variant = V_PUSH_TPV;
        c->phase = PH_FWD;
        c->st_batches += 1;
        c->st_lane_entries += (unsigned long long)lanes;
        if (a.lvl) (void)atomicAdd(&level_of(gc, a, 0).entries, (unsigned long long)cnt);
        const int64_t dp = c->dump_pos;
        c->dump_lane = (dp >= start && dp < end && c->dump_state == 0) ? (int)(dp - start) : -1;
        sf->nf = (float)cnt;
        sf->mf = (float)mf;
        sf->nu = (float)c->range_nodeg;
        sf->mu = (float)c->range_arcs;
        sf->level = 0;
    }
    __syncthreads();
    int lbo;
    const int v = choose_variant(a.p, c->policy, V_PUSH_TPV, *sf, (float)(c->range_hi - c->range_lo),
                                 (float)c->range_arcs, lds, &lbo);
    if (t == 0) set_level_variant(a, c, v, lbo, *sf, (float)(c->range_hi - c->range_lo), (float)c->range_arcs);
}

#ifndef BC_WAVES
#define BC_WAVES 5
#endif
// Register budget of the step kernel: at least BC_WAVES wavefronts per SIMD
// (memory latency is hidden by resident wavefronts; 5 against 6, which spills:
// the damaged 1024^2 grid 102 against 106 ms, R-MAT 18 32.7 against 32.9; 4:
// R-MAT 18 41 against 38.5 with full launches).
//
// A step without work to speak of costs 9.8 us per launch (6.3 in the block engine,
// 7.8 per source) where it cost 21.8 (13.4, 15.9): the state is read and
// written as a whole through LDS instead of field by field, workgroups
// without work leave without counting themselves in, a step of one workgroup
// exchanges no counters, and a level's records are requested together.
// One step of the level state machine for workgroup bid of a launch of
// `grid` workgroups of NW wavefronts: the step kernel below runs it once per
// launch over the whole grid; the block engine runs it in a loop inside one
// workgroup (grid = 1), which then owns the state machine alone, its control block
// gc in LDS (SOLO).
// load() gives the arguments anew to each phase, so that no phase holds
// the others' pointers in its registers.
template <int MODE, int NW, bool SOLO, class Load, class C>
__device__ __forceinline__ void batch_step_body(Load load, C *gc, const int parity, const unsigned bid,
                                                const unsigned grid) {
    constexpr int NT = NW * kWave;
    __shared__ int s_phase, s_level, s_variant, s_last, s_qb, s_qe, s_qn, s_L, s_lo, s_hi, s_dlane, s_cnt;
    __shared__ int s_h0, s_h1, s_hseg, s_hqb, s_gm;
    __shared__ uint32_t s_gb, s_gbn, s_ng;
    __shared__ unsigned s_nblk;
    __shared__ uint32_t s_epoch, s_epoch_b;
    __shared__ unsigned long long s_active, s_dead, s_lmask;
    __shared__ unsigned long long s_red[NW * kNCnt];
    __shared__ unsigned long long s_tot[kNCnt];
    __shared__ unsigned long long s_tmp[kLanes];
    __shared__ int s_lsrc[kLanes];
    __shared__ int s_lead[kLanes];
    __shared__ WaveScratch s_scratch[NW];
    __shared__ StageTotals<NW> s_stot;
    __shared__ float s_lds[2 * kMlpH + kMlpOut + 4];
    __shared__ LevelFeatures s_feat;
    __shared__ float s_il;  // sources-per-entry threshold of this path-count / backward step
    __shared__ int s_usig;  // an undo step restores a path-count step (timing collection)
    __shared__ int s_emax[kLanes], s_emin[kLanes];
    __shared__ Head s_head;
    Head *c = SOLO ? &gc->h[0] : &s_head;
    const int tid = threadIdx.x, lane = tid & 63, wid = uniform(tid >> 6);
    if (!SOLO) {
        head_load<NT>(s_head, gc->h[parity]);
        __syncthreads();
    }
    if (tid == 0) {
        const BatchArgs a = load();
        const int ph = c->phase, l = c->level;
        s_phase = ph;
        s_level = l;
        s_variant = c->variant;
        s_epoch = c->epoch;
        s_epoch_b = c->epoch_b;
        s_active = c->active & ~c->dead;
        s_dead = c->dead;
        s_lmask = c->lane_mask;
        s_L = c->n_levels;
        s_lo = c->range_lo;
        s_hi = c->range_hi;
        s_dlane = c->dump_lane;
        s_usig = c->undo_sig;
        int qb = 0, qe = 0, qn = 0, h0 = 0, h1 = 0, hseg = 0, hqb = 0;
        uint32_t gb = 0, gbn = 0, ng = 0;
        float il = a.p.item_lanes;
        if (ph == PH_FWD || ph == PH_SIG || ph == PH_BWD) {
            // the level's records, requested together: queue offsets, groups, heavy lists
            const int o0 = a.level_off[l], o1 = a.level_off[l + 1], o2 = ph == PH_SIG ? a.level_off[l + 2] : 0;
            const uint32_t g0 = a.gbase[l], g1 = a.gbase[l + 1], g2 = ph == PH_SIG ? a.gbase[l + 2] : 0u;
            const int f0 = a.hq.off[l], f1 = a.hq.off[l + 1], f2 = ph == PH_SIG ? a.hq.off[l + 2] : 0;
            const int ns = a.hq.nseg[ph == PH_SIG ? l + 1 : l];
            const int sel = l < a.max_levels + 2 ? a.lbsel[l] : kLbDefault;
            qb = o0;
            qe = o1;
            qn = o2;
            hqb = f1;   // heavy entries of level l+1 start here
            gbn = g1;   // groups of level l+1 are appended here
            hseg = ns;
            if (ph == PH_SIG) {
                h0 = f1;
                h1 = f2;
                gb = g1;
                ng = g2 - g1 - 1u;
            } else {
                h0 = f0;
                h1 = f1;
                gb = g0;
                ng = g1 - g0 - 1u;
            }
            if (ph != PH_FWD) {
                // the option timed (collection), else the one chosen with level l
                const int opt = c->collect ? c->clb : (ph == PH_SIG ? (sel & 3) : ((sel >> 2) & 3));
                il = lb_item_lanes(a.p, opt);
            } else if (c->variant == V_PULL) {  // static heavy vertices of the batch's range
                h0 = lower_bound_i32(a.g.hv_vtx, a.g.n_heavy, c->range_lo);
                h1 = lower_bound_i32(a.g.hv_vtx, a.g.n_heavy, c->range_hi);
                hseg = a.g.hv_seg[h1] - a.g.hv_seg[h0];
            }
        } else if (ph == PH_DUMP_FWD || ph == PH_DUMP_BWD) {
            qe = a.level_off[c->n_levels];
        } else if (ph == PH_UNDO) {
            qe = a.level_off[l + 1];
            qn = (int)(uint32_t)gc->next_qc;
        }
        // consecutive groups of a large level are taken together (a group
        // costs a wavefront its entries' offsets and words before the first arc)
        const int gm = merge_groups(ng, grid * NW);
        // wavefront work items of this step -> workgroups taking part
        long long items = 1;
        const int cnt = qe - qb;
        if (ph == PH_FWD) {
            if (c->variant == V_PUSH_TPV) items = ((long long)ng + gm - 1) / gm + hseg;
            else if (c->variant == V_PUSH_WPV) items = (long long)cnt + hseg;
            else items = (c->range_hi - c->range_lo + kWave - 1) / kWave + hseg;
        } else if (ph == PH_SIG || ph == PH_BWD) {
            items = ((long long)ng + gm - 1) / gm + hseg;
        } else if (ph == PH_BC) {
            items = (c->range_hi - c->range_lo + kWave - 1) / kWave;
        } else if (ph == PH_DUMP_FWD || ph == PH_DUMP_BWD) {
            items = (qe + kWave - 1) / kWave;
        } else if (ph == PH_UNDO) {
            items = (qn + kWave - 1) / kWave;
        }
        s_nblk = SOLO ? 1u : active_blocks(items, grid);
        s_qb = qb;
        s_qe = qe;
        s_qn = qn;
        s_h0 = h0;
        s_h1 = h1;
        s_hseg = hseg;
        s_hqb = hqb;
        s_gb = gb;
        s_gbn = gbn;
        s_ng = ng;
        s_gm = gm;
        s_il = il;
    }
    if (tid < kLanes) {
        s_emax[tid] = INT_MIN;
        s_emin[tid] = INT_MAX;
    }
    __syncthreads();
    const int phase = uniform(s_phase);
    if (phase == PH_DONE || phase == PH_IDLE) return;
    const unsigned nblk = (unsigned)uniform((int)s_nblk);
    if (bid >= nblk) return;  // no work for this workgroup

    const int gw = (int)bid * NW + wid;
    const int nw = (int)nblk * NW;
    const int l = uniform(s_level);
    const int h0 = uniform(s_h0), h1 = uniform(s_h1), hseg = uniform(s_hseg);

    // (one thread's share of a step fits 32 bits: a level holds a vertex and an
    // arc at most once, spread over the lanes of at least one wavefront)
    unsigned my_edges = 0, my_arcs = 0, my_larcs = 0, my_full_n = 0, my_full_m = 0, my_pairs = 0, my_lent = 0;
    unsigned long long my_act = 0, my_ovf = 0;
    int my_maxe = INT_MIN, my_mine = INT_MAX;

    if (phase == PH_FWD) {
        const BatchArgs a = load();
        const int32_t *__restrict__ rp = a.g.row_ptr;
        const int32_t *__restrict__ col = a.g.col;
        const Tagged *fw_cur = (l & 1) ? a.fw1 : a.fw0;
        const int qb = uniform(s_qb), qe = uniform(s_qe), cnt = qe - qb;
        const uint32_t T = s_epoch + (uint32_t)l;
        const unsigned long long act = uniform(s_active);
        const int variant = uniform(s_variant);
        GroupArgs gr;
        gr.gstart = a.gstart;
        gr.gb = (uint32_t)uniform((int)s_gbn);
        gr.gcap = a.gcap;
        const auto to = stage_to(gc, a.lq_vtx, (uint32_t)qe, a.lq_cap, a.hq, (uint32_t)uniform(s_hqb), gr, a.g,
                                 [&](int w, bool) { return class_deg(a.g, w, rp[w + 1] - rp[w]); });
        Append<decltype(to)> ap{to, s_scratch[wid].w.st, 0};
        Packing &pk = s_scratch[wid].w.pk;
        if (variant == V_PUSH_TPV || variant == V_PUSH_WPV) {
            const int ng = uniform((int)s_ng), gm = uniform(s_gm);
            const uint32_t *gs = a.gstart + uniform((int)s_gb);
            const int n_light = variant == V_PUSH_TPV ? (ng + gm - 1) / gm : cnt;
            const int total = n_light + hseg;
            for (int k = gw; k < total; k += nw) {
                const int it = k < hseg ? n_light + k : k - hseg;  // heavy segments first
                if (it >= n_light) {  // one segment of a heavy frontier vertex
                    const int t = it - n_light;
                    const int h = uniform(seg_owner(a.hq.seg, h0, h1, t));
                    const int s = t - uniform(a.hq.seg[h]);
                    const int p = uniform(a.hq.pos[h]);
                    const int u = uniform(a.lq_vtx[p]);
                    const unsigned long long f = uniform(a.lq_mask[p]) & act;
                    const int a0 = seg_begin(a.g, uniform(rp[u]), s);
                    const int a1 = seg_end(a.g, uniform(rp[u]), uniform(rp[u + 1]), s);
                    if (lane == 0) my_arcs += (unsigned)(a1 - a0);
                    if (f) push_arcs(a, ap, f, a0, a1, col);
                } else if (variant == V_PUSH_WPV) {
                    const int u = uniform(a.lq_vtx[qb + it]);
                    const unsigned long long f = uniform(a.lq_mask[qb + it]) & act;
                    const int e0 = uniform(rp[u]), e1 = uniform(rp[u + 1]);
                    if (!f || uniform(class_deg(a.g, u, e1 - e0)) > seg_arcs(a.g)) continue;  // heavy ones run as segments
                    if (lane == 0) my_arcs += (unsigned)(e1 - e0);
                    push_arcs(a, ap, f, e0, e1, col);
                } else {  // a group of frontier vertices per wavefront
                    const int i0 = uniform((int)gs[it * gm]), i1 = min(uniform((int)gs[min(it * gm + gm, ng)]), cnt);
                    if (i1 > i0) my_arcs += push_group(a, ap, pk, qb, i0, i1, act, rp, col);
                }
            }
        } else {  // V_PULL over the batch's vertex range, scanning in-arcs (predecessors)
            const int32_t *__restrict__ irp = a.g.in_row_ptr;
            const int32_t *__restrict__ icol = a.g.in_col;
            const int lo = uniform(s_lo), span = uniform(s_hi) - lo;
            const int n_light = (span + kWave - 1) / kWave;
            const int total = n_light + hseg;
            const int hs0 = uniform(a.g.hv_seg[h0]);
            for (int k = gw; k < total; k += nw) {
                const int it = k < hseg ? n_light + k : k - hseg;  // heavy segments first
                if (it >= n_light) {  // one segment of a heavy unvisited vertex
                    const int t = hs0 + (it - n_light);
                    const int h = uniform(seg_owner(a.g.hv_seg, h0, h1, t));
                    const int s = t - uniform(a.g.hv_seg[h]);
                    const int w = uniform(a.g.hv_vtx[h]);
                    const unsigned long long need = act & ~uniform(a.vn[w].vis);
                    const int a0 = seg_begin(a.g, uniform(irp[w]), s);
                    const int a1 = seg_end(a.g, uniform(irp[w]), uniform(irp[w + 1]), s);
                    int scanned = 0;
                    const unsigned long long got = pull_arcs(fw_cur, T, need, a0, a1, icol, scanned);
                    if (lane == 0) my_arcs += (unsigned)scanned;
                    bool newly = false;
                    if (lane == 0 && got) newly = atomicOr(&a.vn[w].nxt, got) == 0ull;
                    append(ap, newly, w);
                    continue;
                }
                // runs of 2^pull_log consecutive vertices from all over the range
                const int i = (((lane >> a.g.pull_log) * n_light + it) << a.g.pull_log) + (lane & ((1 << a.g.pull_log) - 1));
                const int w = lo + i;
                const bool valid = i < span;
                const unsigned long long vis = valid ? a.vn[w].vis : ~0ull;
                const unsigned long long need = act & ~vis;
                const int e0 = need ? irp[w] : 0;
                const int ni = need ? irp[w + 1] - e0 : 0;  // in-arcs to scan
                const int od = (need && a.g.directed) ? rp[w + 1] - rp[w] : ni;
                const int deg = a.g.directed ? max(ni, od) : ni;  // class degree
                const int len = deg <= kLightDeg ? ni : 0;
                unsigned long long got = 0;
                int scanned = 0;
                // one thread per vertex, four arcs at a time
                for (int t = 0; __any(t < len && got != need); t += 4) {
                    if (t < len && got != need) {
                        int u[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) u[q] = icol[e0 + min(t + q, len - 1)];
                        unsigned long long g4 = 0;
#pragma unroll
                        for (int q = 0; q < 4; ++q) g4 |= tagged_lanes(fw_cur, u[q], T, need);
                        got |= g4;
                        scanned += min(4, len - t);
                    }
                }
                // medium-degree vertices: the whole wavefront, one at a time
                for (unsigned long long mm = __ballot(deg > kLightDeg && deg <= seg_arcs(a.g)); mm; mm &= mm - 1) {
                    const int j = __ffsll(mm) - 1;
                    const int m0 = __builtin_amdgcn_readlane(e0, j), m1 = m0 + __builtin_amdgcn_readlane(ni, j);
                    int sc = 0;
                    const unsigned long long gj = pull_arcs(fw_cur, T, readlane_u64(need, j), m0, m1, icol, sc);
                    if (lane == 0) scanned += sc;
                    if (lane == j) got = gj;
                }
                my_arcs += (unsigned)scanned;
                const bool found = got != 0ull && deg <= seg_arcs(a.g);
                if (found) a.vn[w].nxt = got;
                append(ap, found, w);
            }
        }
        stage_finish<NW>(ap.st, ap.n, s_stot, to);
    } else if (phase == PH_SIG) {
        const BatchArgs a = load();
        const int32_t *__restrict__ rp = a.g.row_ptr;
        Tagged *fw_cur = (l & 1) ? a.fw1 : a.fw0, *fw_nxt = (l & 1) ? a.fw0 : a.fw1;
        // path counts of the new level; lane = source
        const int qs = uniform(s_qe), cnt = uniform(s_qn) - qs;
        const uint32_t T = s_epoch + (uint32_t)l;
        const int sh = MODE ? a.shift[(size_t)l * kLanes + lane] : 0;
        const unsigned long long lmask = s_lmask;
        const int ng = uniform((int)s_ng), gm = uniform(s_gm), n_groups = (ng + gm - 1) / gm;
        const uint32_t *gs = a.gstart + uniform((int)s_gb);
        const int total = n_groups + hseg;
        const float il = s_il;
        constexpr int OP = MODE ? OP_F64 : OP_U64;
        Packing &pk = s_scratch[wid].w.pk;
        SigCounters sc;
        for (WorkCursor<NW> wc(gc, nblk, bid); wc.item() < total; wc.next(total)) {
            const int k = wc.item();
            const int it = k < hseg ? n_groups + k : k - hseg;  // heavy segments first
            if (it < n_groups) {
                const int i0 = uniform((int)gs[it * gm]), i1 = min(uniform((int)gs[min(it * gm + gm, ng)]), cnt);
                if (i1 > i0) sig_group<MODE>(a, fw_cur, fw_nxt, T, qs, i0, i1, sh, lmask, sc, l, s_emax, s_emin, il, pk);
                continue;
            }
            // a segment of a heavy new vertex
            const int t = it - n_groups;
            const int h = uniform(seg_owner(a.hq.seg, h0, h1, t));
            const int s0 = uniform(a.hq.seg[h]), s = t - s0;
            const int p = uniform(a.hq.pos[h]);
            const int w = uniform(a.lq_vtx[p]);
            const int e0 = uniform(a.g.in_row_ptr[w]), e1 = uniform(a.g.in_row_ptr[w + 1]);  // predecessors: in-arcs
            const int od = uniform(rp[w + 1] - rp[w]);
            const unsigned long long m = uniform(a.vn[w].nxt);
            const int a0 = seg_begin(a.g, e0, s), a1 = seg_end(a.g, e0, e1, s);
            RowSum<OP> sum;
            row_arcs<OP>(TagLanes{fw_cur, T}, m, a0, a1, sh, a.g.in_col, a.sigma, sum, sc.ac);
            const size_t slot = (size_t)(s0 + s) * kLanes + lane;
            if (MODE == 0) {
                part_store(&a.hq.part_lo[slot], sum.lo);
                part_store(&a.hq.part_hi[slot], sum.hi);
            } else {
                part_store(&a.hq.part_lo[slot], as_u64(sum.d));
            }
            const int ns = n_segments(a.g, uniform(class_deg(a.g, w, od)));
            if (!seg_arrive(&a.hq.cnt[h], ns)) continue;
            sum.clear();
            for (int k2 = 0; k2 < ns; ++k2) {  // combine in segment order
                const size_t sl = (size_t)(s0 + k2) * kLanes + lane;
                if (MODE == 0) {
                    sum.add(part_load(&a.hq.part_lo[sl]), 0);
                    sum.hi += (unsigned)part_load(&a.hq.part_hi[sl]);
                } else {
                    sum.d += as_f64(part_load(&a.hq.part_lo[sl]));
                }
            }
            if (lane == 0) a.hq.cnt[h] = 0;
            const VisNext x = a.vn[w];
            unsigned long long ovf = 0;
            sig_store<OP>(sum, m, row_addr(a.sigma, w), a.sigma_limit, ovf, sc);
            sc.ovf |= ovf;
            if (lane == 0) sig_publish(a, fw_nxt, T + 1u, p, w, x.vis, x.nxt, od, lmask, sc);
        }
        my_edges += sc.edges;
        my_act |= sc.act;
        my_ovf |= sc.ovf;
        my_full_n += sc.full_n;
        my_full_m += sc.full_m;
        my_larcs += sc.ac.larcs;
        my_arcs += sc.ac.arcs;
        my_pairs += sc.ac.pairs;
        my_lent += sc.lent;
        my_maxe = max(my_maxe, sc.maxe);
        my_mine = min(my_mine, sc.mine);
    } else if (phase == PH_BWD) {
        const BatchArgs a = load();
        const int32_t *__restrict__ rp = a.g.row_ptr;
        const int32_t *__restrict__ col = a.g.col;
        Tagged *fw_cur = (l & 1) ? a.fw1 : a.fw0, *fw_nxt = (l & 1) ? a.fw0 : a.fw1;
        const int qb = s_qb, cnt = s_qe - s_qb;
        const uint32_t TB = s_epoch_b + (uint32_t)l;
        Tagged *fb_cur = fw_cur;  // written with this level's tag
        Tagged *fb_nxt = fw_nxt;  // read: level l+1's tag
        const unsigned long long dead = uniform(s_dead);
        const int sh = MODE ? a.shift[(size_t)l * kLanes + lane] : 0;
        const int shn = (MODE && l + 1 < s_L) ? a.shift[(size_t)(l + 1) * kLanes + lane] : 0;
        const int ng = uniform((int)s_ng), gm = uniform(s_gm), n_groups = (ng + gm - 1) / gm;
        const uint32_t *gs = a.gstart + uniform((int)s_gb);
        const int total = n_groups + hseg;
        const bool has_next = l + 1 < uniform(s_L);
        const float il = s_il;
        Packing &pk = s_scratch[wid].w.pk;
        ArcCounters ac;
        for (WorkCursor<NW> wc(gc, nblk, bid); wc.item() < total; wc.next(total)) {
            const int k = wc.item();
            const int it = k < hseg ? n_groups + k : k - hseg;  // heavy segments first
            if (it < n_groups) {
                const int i0 = uniform((int)gs[it * gm]), i1 = min(uniform((int)gs[min(it * gm + gm, ng)]), cnt);
                if (i1 > i0) bwd_group<MODE>(a, fb_nxt, fb_cur, TB, qb, i0, i1, dead, sh, shn, ac, l, has_next, il, pk);
                continue;
            }
            const int t = it - n_groups;
            const int h = uniform(seg_owner(a.hq.seg, h0, h1, t));
            const int s0 = uniform(a.hq.seg[h]), s = t - s0;
            const int p = uniform(a.hq.pos[h]);
            const int v = uniform(a.lq_vtx[p]);
            const unsigned long long Mf = uniform(a.lq_mask[p]);
            const unsigned long long M = Mf & ~dead;
            const int e0 = uniform(rp[v]), e1 = uniform(rp[v + 1]);  // successors: out-arcs
            const int a0 = seg_begin(a.g, e0, s), a1 = seg_end(a.g, e0, e1, s);
            RowSum<OP_C> sum;
            if (M) row_arcs<OP_C>(TagLanes{fb_nxt, TB + 1u}, M, a0, a1, 0, col, a.chat, sum, ac);
            part_store(&a.hq.part_lo[(size_t)(s0 + s) * kLanes + lane], as_u64(sum.d));
            const int ns = n_segments(a.g, uniform(class_deg(a.g, v, e1 - e0)));
            if (!seg_arrive(&a.hq.cnt[h], ns)) continue;
            double acc = 0.0;
            for (int k2 = 0; k2 < ns; ++k2) acc += as_f64(part_load(&a.hq.part_lo[(size_t)(s0 + k2) * kLanes + lane]));
            if (lane == 0) a.hq.cnt[h] = 0;
            const unsigned slot = row_slot(M);
            double delta, cc;
            bwd_values<MODE>(row_load(row_addr(a.sigma, v), slot), acc, sh, shn, delta, cc);
            row_store(row_addr(a.chat, v), slot, as_u64(cc));
            row_store(row_addr(a.delta, v), slot, as_u64(delta));
            if (lane == 0) {
                Tagged tg;
                tg.mask = Mf;
                tg.tag = TB;
                fb_cur[v] = tg;
            }
        }
        my_larcs += ac.larcs;
        my_arcs += ac.arcs;
        my_pairs += ac.pairs;
    } else if (phase == PH_UNDO) {
        const BatchArgs a = load();
        const int qs = s_qe, cnt = s_qn;
        if (s_usig) {
            // timing collection: the entries of level l+1 get back the words
            // they had before their path-count step (that step set the lanes
            // of their queue masks visited and cleared their next words)
            for (int i = (int)bid * NT + tid; i < cnt; i += (int)nblk * NT) {
                const int w = a.lq_vtx[qs + i];
                const unsigned long long m = a.lq_mask[qs + i];
                VisNext x = a.vn[w];
                x.vis &= ~m;
                x.nxt = m;
                a.vn[w] = x;
            }
        } else {
            // timing collection: forget the level just discovered (its
            // entries are the only vertices with next words set)
            for (int i = (int)bid * NT + tid; i < cnt; i += (int)nblk * NT) a.vn[a.lq_vtx[qs + i]].nxt = 0ull;
        }
    } else if (phase == PH_BC) {
        const BatchArgs a = load();
        if (tid < kLanes) s_lsrc[tid] = a.lane_src[tid];
        __syncthreads();
        // dependencies -> BC in lane order (the run's source order), then
        // clear the visited words.  A wavefront takes 64 consecutive
        // vertices; their delta rows are read 8 lanes (64 bytes) at a time,
        // 8 rows per load (coalesced), staged through LDS, and each vertex's
        // own thread adds its lanes in ascending order (a source's own lane
        // and lanes not reached are skipped: they would add +0.0, which
        // leaves the non-negative sum's bits unchanged)
        const int lo = s_lo, span = s_hi - s_lo;
        const unsigned long long keep = s_lmask & ~s_dead;
        const int wv = wid;
        double *tile = s_scratch[wv].tile;
        for (int base = ((int)bid * NW + wv) * kWave; base < span; base += (int)nblk * NT) {
            const int i = base + lane;
            const int w = lo + i;
            VisNext x;
            x.vis = 0ull;
            x.nxt = 0ull;
            if (i < span) x = a.vn[w];
            const unsigned long long vis = x.vis & keep;
            if (__ballot(vis != 0ull)) {
                double b = vis ? a.bc[w] : 0.0;
                for (int c = 0; c < kLanes / 8; ++c) {
                    const unsigned m8 = (unsigned)(vis >> (8 * c)) & 0xFFu;
                    if (!__ballot(m8 != 0u)) continue;
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const int vi = 8 * r + (lane >> 3);  // vertex of the 64 whose row this lane reads
                        const int kk = lane & 7;
                        const unsigned mv = (unsigned)__shfl((int)m8, vi);
                        double d = 0.0;
                        if ((mv >> kk) & 1u) d = a.delta[(size_t)(lo + base + vi) * kLanes + 8 * c + kk];
                        tile[vi * 8 + (kk ^ (vi & 7))] = d;
                    }
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        if (((m8 >> j) & 1u) && s_lsrc[8 * c + j] != w) b += tile[lane * 8 + (j ^ (lane & 7))];
                    }
                    __builtin_amdgcn_wave_barrier();
                }
                if (vis) a.bc[w] = b;
            }
            if (x.vis | x.nxt) {
                VisNext z;
                z.vis = 0ull;
                z.nxt = 0ull;
                a.vn[w] = z;
            }
        }
    } else if (phase == PH_DUMP_FWD || phase == PH_DUMP_BWD) {
        const BatchArgs a = load();
        const int k = s_dlane;
        const int L = s_L;
        const int total = s_qe;
        for (int j = (int)bid * NT + tid; j < total; j += (int)nblk * NT) {
            if (!((a.lq_mask[j] >> k) & 1ull)) continue;
            int lo = 0, hi = L;  // level of entry j: level_off[lvl] <= j < level_off[lvl+1]
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (a.level_off[mid] <= j) lo = mid;
                else hi = mid;
            }
            const int v = a.lq_vtx[j];
            if (phase == PH_DUMP_FWD) {
                a.dump_d[v] = lo;
                a.dump_sig[v] = a.sigma[(size_t)v * kLanes + k];
            } else if (lo >= 1) {
                a.dump_delta[v] = a.delta[(size_t)v * kLanes + k];
            }
        }
        if (phase == PH_DUMP_FWD && bid == 0)
            for (int i = tid; i < L; i += NT) a.dump_shift[i] = MODE ? a.shift[(size_t)i * kLanes + k] : 0;
    }

    // ---- per-launch counters into the slots; the last workgroup continues
    Counters cn;
    cn.v[SC_EDGES] = my_edges;
    cn.v[SC_ARCS] = my_arcs;
    cn.v[SC_LARCS] = my_larcs;
    cn.v[SC_FULLN] = my_full_n;
    cn.v[SC_FULLM] = my_full_m;
    cn.v[SC_ACT] = my_act;
    cn.v[SC_OVF] = my_ovf;
    cn.v[SC_PAIRS] = my_pairs;
    cn.v[SC_LENT] = my_lent;
    const BatchArgs a = load();
    if (MODE == 1 && phase == PH_SIG) {
        // per-lane exponent range of the new level: reduced over the
        // workgroup in LDS, then one atomic per lane into the workgroup's slot
        if (my_maxe != INT_MIN) atomicMax(&s_emax[lane], my_maxe);
        if (my_mine != INT_MAX) atomicMin(&s_emin[lane], my_mine);
        __syncthreads();
        if (nblk > 1) {
            const int slot = (int)(bid % kSlots);
            if (tid < kLanes && s_emax[tid] != INT_MIN) atomicMax(&a.maxexp[slot * kLanes + tid], s_emax[tid]);
            else if (tid >= kLanes && tid < 2 * kLanes && s_emin[tid - kLanes] != INT_MAX)
                atomicMin(&a.maxexp[(kSlots + slot) * kLanes + tid - kLanes], s_emin[tid - kLanes]);
            // completed before this workgroup arrives (the last one reads them)
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_s_waitcnt(0);
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
        }
    }
    const float *mlp = c->policy == POL_MLP && phase == PH_SIG ? load().p.mlp : nullptr;
    if (!step_epilogue<NW>(gc, cn, s_red, s_tot, &s_last, bid, nblk, mlp)) return;

    // ---- the last workgroup advances the state machine
    int action = 0;  // 1 = begin batch, 2 = advance level
    if (tid == 0) {
        c->st_steps += 1;
        c->st_arcs += s_tot[SC_ARCS];
        c->st_lane_arcs += s_tot[SC_LARCS];
        c->st_lane_entries += s_tot[SC_LENT];
        c->st_parcs[phase] += s_tot[SC_ARCS];
        c->st_plarcs[phase] += s_tot[SC_LARCS];
        c->st_ppairs[phase] += s_tot[SC_PAIRS];
        const unsigned long long now = wall_clock64();
        const unsigned long long prev_tick = c->last_tick;
        const unsigned long long dt = prev_tick ? now - prev_tick : 0ull;
        c->st_ticks[phase] += dt;
        if (phase == PH_FWD) c->st_vticks[s_variant] += dt;
        c->last_tick = now;
        const int rl = (phase == PH_FWD || phase == PH_BWD) ? l : (phase == PH_SIG ? l + 1 : -1);
        if (rl >= 0 && a.lvl) {  // (atomics that nothing waits for)
            LevelRec &r = level_of(gc, a, rl);
            (void)atomicAdd(&r.arcs, s_tot[SC_ARCS]);
            (void)atomicAdd(&r.ticks, dt);
            if (phase == PH_FWD) {
                (void)atomicAdd(&r.visits, 1ull);
                (void)atomicAdd(&r.var[s_variant], 1ull);
            }
        }
        bool timed_again = false;
        // one training sample: features x, device ticks t[0..2] at outputs k0..k0+2
        auto put_sample = [&](const float *x, const unsigned long long *t, int k0) {
            const uint32_t k = c->n_samples;
            if (k < a.col_cap) {
                for (int i = 0; i < kMlpIn; ++i) a.col_X[(size_t)k * kMlpIn + i] = x[i];
                for (int j = 0; j < kMlpOut; ++j)
                    a.col_Y[(size_t)k * kMlpOut + j] = (j >= k0 && j < k0 + 3) ? (float)t[j - k0] : -1.0f;
            }
            c->n_samples = k + 1;
        };
        if (phase == PH_FWD && c->collect) {
            c->ct[c->cvar] = c->last_tick ? now - prev_tick : 0ull;
            if (c->cvar < 2) {
                timed_again = true;  // undo, then run the level with the next variant
                c->phase = PH_UNDO;
                c->undo_sig = 0;
            } else {
                put_sample(c->feat, c->ct, kOutFwd);
                c->cvar = 0;
            }
        }
        if (phase == PH_SIG && c->collect) {
            // the path counts of level l+1 under each summation option (the
            // features are those of level l, which chose the option)
            c->ct_lb[c->clb] = dt;
            if (c->clb < 2) {
                timed_again = true;  // restore the level's words, then sum again
                c->phase = PH_UNDO;
                c->undo_sig = 1;
            } else {
                if (a.col_F && l < a.max_levels + 2) put_sample(a.col_F + (size_t)l * kMlpIn, c->ct_lb, kOutSig);
                c->clb = 0;
            }
        }
        if (phase == PH_BWD && c->collect) {
            // the backward step overwrites what it writes: run it again as is
            c->ct_lb[c->clb] = dt;
            if (c->clb < 2) {
                timed_again = true;
                c->clb += 1;
            } else {
                if (a.col_F && l < a.max_levels + 2) put_sample(a.col_F + (size_t)l * kMlpIn, c->ct_lb, kOutBwd);
                c->clb = 0;
            }
        }
        if (phase == PH_UNDO && c->undo_sig) {
            c->undo_sig = 0;
            c->clb += 1;
            c->phase = PH_SIG;
        } else if (phase == PH_UNDO) {
            gc->next_qc = 0ull;
            gc->next_hq = 0;
            c->cvar += 1;
            c->variant = c->cvar;
            c->phase = PH_FWD;
        } else if (timed_again) {
        } else if (phase == PH_FWD) {
            const unsigned long long qc = ld_agent(&gc->next_qc);
            const uint32_t cnt = (uint32_t)qc, cost = (uint32_t)(qc >> 32);
            const unsigned long long nh = ld_agent(&gc->next_hq);
            const int qe = s_qe;  // level_off[l + 1]
            c->st_fwd_levels += 1;
            c->st_var[s_variant] += 1;
            c->st_qentries += cnt;
            if (a.lvl) (void)atomicAdd(&level_of(gc, a, l + 1).entries, (unsigned long long)cnt);
            a.hq.off[l + 2] = s_hqb + (int)(uint32_t)nh;
            a.hq.nseg[l + 1] = (int)(nh >> 32);
            gc->next_hq = 0;
            if (cnt == 0) {
                const int L = l + 1;
                c->n_levels = L;
                if (MODE == 1 && c->f64_check) {
                    // counts below 2^65 might fit in 64 bits: hand the lane back
                    // (no contribution here), a 64-bit pass decides its mode
                    unsigned long long back = 0;
                    for (int k = 0; k < kLanes; ++k)
                        if (c->lane_emax[k] <= 65) back |= 1ull << k;
                    back &= c->lane_mask & ~c->dead;
                    const int64_t start = a.batch_start[c->pos];
                    for (unsigned long long o = back; o; o &= o - 1) {
                        const int k = __ffsll(o) - 1;
                        const uint32_t q = c->n_ovf;
                        if (q < a.ovf_cap) a.ovf_list[q] = start + k;
                        else gc->err |= ERR_OVF_CAP;
                        c->n_ovf = q + 1;
                    }
                    c->dead |= back;
                }
                // backward tags epoch_b + 1 .. epoch_b + L lie above every forward tag
                c->epoch_b = c->epoch + (uint32_t)L + 1u;
                if ((unsigned long long)L > c->st_max_levels) c->st_max_levels = L;
                if (c->dump_lane >= 0 && !((c->dead >> c->dump_lane) & 1ull)) c->phase = PH_DUMP_FWD;
                else if (L >= 2) { c->phase = PH_BWD; c->level = L - 1; }
                else c->phase = PH_BC;
            } else if (l + 2 >= a.max_levels) {
                gc->err |= ERR_LEVEL_CAP;
                c->phase = PH_DONE;
            } else {
                a.level_off[l + 2] = qe + (int)cnt;
                // close the groups of level l+1 (every entry costs >= 2 units)
                const uint32_t gb = s_gbn;  // gbase[l + 1]
                const uint32_t ng = (cost - 1u) / (uint32_t)kBudget + 1u;
                if ((unsigned long long)gb + ng + 1u > a.gcap) {
                    gc->err |= ERR_QUEUE_CAP;
                    c->phase = PH_DONE;
                } else {
                    a.gstart[gb] = 0u;
                    a.gstart[gb + ng] = cnt;
                    a.gbase[l + 2] = gb + ng + 1u;
                    c->phase = PH_SIG;
                }
            }
        } else if (phase == PH_SIG) {
            action = 2;
        } else if (phase == PH_BWD) {
            if (l - 1 >= 1) {
                c->level = l - 1;
            } else if (c->dump_lane >= 0 && c->dump_state == 1) {
                c->phase = PH_DUMP_BWD;
            } else {
                c->phase = PH_BC;
            }
        } else if (phase == PH_DUMP_FWD) {
            c->dump_state = 1;
            const int L = c->n_levels;
            if (L >= 2) { c->phase = PH_BWD; c->level = L - 1; }
            else c->phase = PH_DUMP_BWD;
        } else if (phase == PH_DUMP_BWD) {
            c->dump_state = 2;
            c->phase = PH_BC;
        } else if (phase == PH_BC) {
            // the next batch is set up by the last workgroup of a launch of
            // its own: this launch's workgroups have just cleared visited
            // words that the set-up writes again
            const int64_t next = c->pos + 1;
            c->pos = next;
            c->phase = next < c->n_items ? PH_FIN : PH_DONE;
        } else if (phase == PH_FIN) {
            action = 1;
        }
        s_cnt = action;
    }
    __syncthreads();
    action = s_cnt;
    if (action == 1) {
        gc->next_qc = 0ull;
        gc->next_hq = 0ull;
        batch_begin<MODE>(a, gc, c, c->pos, s_lds, &s_feat, s_lsrc, &s_qn, s_tmp, s_lead);
    } else if (action == 2) {
        // finish level l+1: lane deaths, FP64 shifts, features, policy
        if (tid == 0) {
            const unsigned long long ovf = s_tot[SC_OVF] & ~c->dead;
            if (ovf) {
                unsigned long long o = ovf;
                const int64_t start = a.batch_start[c->pos];
                while (o) {
                    const int k = __ffsll(o) - 1;
                    o &= o - 1;
                    const uint32_t q = c->n_ovf;
                    if (q < a.ovf_cap) a.ovf_list[q] = start + k;
                    else gc->err |= ERR_OVF_CAP;
                    c->n_ovf = q + 1;
                }
                c->dead |= ovf;
            }
            c->active = s_tot[SC_ACT] & ~c->dead;
        }
        if (MODE && nblk > 1) {
            // exponent ranges of the workgroups: all slots read at once
            constexpr int kPer = kSlots / NW;
            const int nslots = (int)min(nblk, (unsigned)kSlots);
            int mx[kPer], mn[kPer];
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int sl = wid + q * NW;
                mx[q] = sl < nslots ? ld_agent(&a.maxexp[sl * kLanes + lane]) : INT_MIN;
                mn[q] = sl < nslots ? ld_agent(&a.maxexp[(kSlots + sl) * kLanes + lane]) : INT_MAX;
            }
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int sl = wid + q * NW;
                if (sl >= nslots) break;
                atomicMax(&s_emax[lane], mx[q]);
                atomicMin(&s_emin[lane], mn[q]);
                a.maxexp[sl * kLanes + lane] = INT_MIN;
                a.maxexp[(kSlots + sl) * kLanes + lane] = INT_MAX;
            }
            __syncthreads();
        }
        if (MODE && tid < kLanes) {
            const int mx = s_emax[tid], mn = s_emin[tid];
            int sh = 0;
            if (mx != INT_MIN && mx > kExpHigh) sh = mx - kExpTarget;
            if (mn != INT_MAX && mn - sh < kExpLow) atomicOr(&gc->err, ERR_SIGMA_RANGE);
            a.shift[(size_t)(l + 1) * kLanes + tid] = sh;
            // true counts of level l+1 are the stored ones times 2^lane_E
            if (mx != INT_MIN) c->lane_emax[tid] = max(c->lane_emax[tid], mx + c->lane_E[tid]);
            c->lane_E[tid] += sh;
        }
        if (tid == 0) {
            const uint32_t cnt = (uint32_t)ld_agent(&gc->next_qc);
            const unsigned long long edges = s_tot[SC_EDGES];
            c->level = l + 1;
            c->visited_n += cnt;
            c->visited_m += edges;
            c->full_n += s_tot[SC_FULLN];
            c->full_m += s_tot[SC_FULLM];
            const unsigned long long fn = c->full_n, fm = c->full_m;
            s_feat.nf = (float)cnt;
            s_feat.mf = (float)edges;
            s_feat.nu = (float)((long long)c->range_nodeg - (long long)fn);
            s_feat.mu = (float)((long long)c->range_arcs - (long long)fm);
            s_feat.level = l + 1;
            gc->next_qc = 0ull;
            c->prev_variant = c->variant;
            c->phase = PH_FWD;
        }
        __syncthreads();
        int lbo;
        const int v = choose_variant(a.p, c->policy, c->prev_variant, s_feat, (float)(c->range_hi - c->range_lo),
                                     (float)c->range_arcs, s_lds, &lbo);
        if (tid == 0)
            set_level_variant(a, c, v, lbo, s_feat, (float)(c->range_hi - c->range_lo), (float)c->range_arcs);
    }
    if constexpr (!SOLO) head_store(gc, s_head, parity);
}

// Arguments of a step launch, read from the kernel's own argument segment.
struct LaunchArgs {
    typedef const __attribute__((address_space(4))) unsigned long long *Words;
    Words p;
    __device__ __forceinline__ LaunchArgs() : p((Words)__builtin_amdgcn_kernarg_segment_ptr()) {}
    __device__ __forceinline__ BatchArgs operator()() const {
        Words q = p;
        asm volatile("" : "+s"(q));  // the loads stay in the phase that asks
        BatchArgs a;
        static_assert(sizeof(BatchArgs) % 8 == 0, "copied in 8-byte words");
        unsigned long long *d = (unsigned long long *)&a;
#pragma unroll
        for (int i = 0; i < (int)(sizeof(BatchArgs) / 8); ++i) d[i] = q[i];
        return a;
    }
};

template <int MODE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(BC_WAVES))) void batch_step(BatchArgs) {
    const LaunchArgs load;
    const BatchArgs a = load();
    batch_step_body<MODE, kWavesPerBlock, false>(load, a.ctl, a.parity, blockIdx.x, gridDim.x);
}

template __global__ void batch_step<0>(BatchArgs);
template __global__ void batch_step<1>(BatchArgs);

// Block engine: a persistent launch in which every workgroup owns a level
// state machine.  A workgroup takes a chunk (batches [b0, b1) of one graph
// with vertices [lo, hi)), points the per-vertex arrays of its arguments at
// its private scratch shifted by lo (every index the steps use lies in
// [lo, hi): arcs never leave a graph), and runs the steps of the chunk one
// after another with workgroup barriers in between.  Scores of the chunk go
// to its own partial vector.  The control block keeps its tag epochs from
// chunk to chunk, so tags left by an earlier chunk never match.  Exit: the
// work queue runs dry (every workgroup takes chunks until the counter passes
// n_chunks), a step reports an error, or a chunk exceeds max_steps per batch.
// Arguments that sit in LDS, moved to scalar registers.
struct LdsArgs {
    const BatchArgs *p;
    __device__ __forceinline__ BatchArgs operator()() const {
        BatchArgs a;
        int *d = (int *)&a;
        const int *q = (const int *)p;
#pragma unroll
        for (int i = 0; i < (int)(sizeof(BatchArgs) / 4); ++i) d[i] = uniform(q[i]);
        return a;
    }
};

template <int MODE, int NW>
__global__ __launch_bounds__(NW * kWave) void block_run(BlockArgs ra) {
    constexpr int NT = NW * kWave;
    // the workgroup's arguments live in LDS: thread 0 points them at the
    // chunk's state, every thread reads them there
    __shared__ BatchArgs s_a;
    __shared__ int s_go;
    const int tid = threadIdx.x;
    // the control block, too: its fields change every step
    __shared__ SoloCtl s_ctl;
    Head *c = &s_ctl.h[0];
    {
        const Head &g = ra.states[blockIdx.x].h;
        for (int i = tid; i < (int)(sizeof(Head) / 8); i += NT)
            ((unsigned long long *)c)[i] = ((const unsigned long long *)&g)[i];
        if (tid == 0) {
            s_ctl.err = 0;
            s_ctl.next_qc = 0ull;
            s_ctl.next_hq = 0ull;
            s_ctl.work[0][0] = 0u;
        }
        static_assert(sizeof(LevelRec) == 64, "taken in 8-byte words");
        for (int i = tid; i < kSoloLevels * 8; i += NT) ((unsigned long long *)s_ctl.lvl)[i] = 0ull;
    }
    char *base = ra.scratch + (size_t)blockIdx.x * ra.stride;
    const BlockLayout L((size_t)ra.nmax, ra.lq_cap, (size_t)ra.max_levels, ra.gcap, ra.hq_entries, ra.hq_levels,
                        ra.part_cap, ra.ovf_cap);
    if (tid == 0) {
        BatchArgs &a = s_a;
        a = ra.a;
        a.ctl = nullptr;
        a.lq_vtx = (int32_t *)(base + L.lq_vtx);
        a.lq_mask = (unsigned long long *)(base + L.lq_mask);
        a.lq_cap = ra.lq_cap;
        a.level_off = (int32_t *)(base + L.level_off);
        a.max_levels = ra.max_levels;
        a.gstart = (uint32_t *)(base + L.gstart);
        a.gbase = (uint32_t *)(base + L.gbase);
        a.lbsel = (int32_t *)(a.gbase + ra.max_levels + 2);
        a.gcap = ra.gcap;
        a.shift = (int32_t *)(base + L.shift);
        a.maxexp = (int32_t *)(base + L.maxexp);
        a.lane_src = (int32_t *)(base + L.lane_src);
        a.hq.pos = (int32_t *)(base + L.hq_pos);
        a.hq.seg = (int32_t *)(base + L.hq_seg);
        a.hq.cnt = (int32_t *)(base + L.hq_cnt);
        a.hq.off = (int32_t *)(base + L.hq_off);
        a.hq.nseg = (int32_t *)(base + L.hq_nseg);
        a.hq.cap = ra.hq_entries;
        a.hq.part_lo = (unsigned long long *)(base + L.part_lo);
        a.hq.part_hi = (unsigned long long *)(base + L.part_hi);
        a.hq.part_cap = ra.part_cap;
        a.ovf_list = (int64_t *)(base + L.ovf);
        a.ovf_cap = ra.ovf_cap;
        a.dump_d = nullptr;
        a.dump_sig = nullptr;
        a.dump_delta = nullptr;
        a.dump_shift = nullptr;
        a.col_X = nullptr;
        a.col_Y = nullptr;
        a.col_cap = 0;
    }
    int32_t *mx = (int32_t *)(base + L.maxexp);
    for (int i = tid; i < 2 * kSlots * kLanes; i += NT) mx[i] = i < kSlots * kLanes ? INT_MIN : INT_MAX;
    for (;;) {
        __syncthreads();
        if (tid == 0) {
            const uint32_t k = atomicAdd(ra.next, 1u);
            const int t = (k < (uint32_t)ra.n_chunks && s_ctl.err == 0) ? ra.order[k] : -1;
            s_go = t;
            if (t >= 0) {
                const int b0 = ra.c_b0[t], b1 = ra.c_b1[t];
                const int lo = ra.a.batch_lo[b0], hi = ra.a.batch_hi[b0];
                BatchArgs &a = s_a;
                a.vn = (VisNext *)(base + L.vn) - lo;
                a.fw0 = (Tagged *)(base + L.fw0) - lo;
                a.fw1 = (Tagged *)(base + L.fw1) - lo;
                a.sigma = (unsigned long long *)(base + L.sigma) - (size_t)lo * kLanes;
                a.chat = (double *)(base + L.chat) - (size_t)lo * kLanes;
                a.delta = (double *)(base + L.delta) - (size_t)lo * kLanes;
                a.bc = ra.partials + ra.c_part[t] - lo;
                // the first step (phase BC of an empty batch) clears the
                // visited words of [lo, hi), then the chunk's batches follow
                c->phase = PH_BC;
                c->pos = (int64_t)b0 - 1;
                c->n_items = b1;
                c->range_lo = lo;
                c->range_hi = hi;
                c->lane_mask = 0ull;
                c->dead = 0ull;
                c->active = 0ull;
                c->level = 0;
            }
        }
        __syncthreads();
        const int t = s_go;
        if (t < 0) break;
        const int b0 = ra.c_b0[t], b1 = ra.c_b1[t];
        const int lo = ra.a.batch_lo[b0], hi = ra.a.batch_hi[b0];
        double *part = ra.partials + ra.c_part[t];
        for (int i = tid; i < hi - lo; i += NT) part[i] = 0.0;
        const int64_t max_steps = (int64_t)(b1 - b0 + 1) * ra.max_steps;
        for (int64_t step = 0;; ++step) {
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (tid == 0) {
                int go = (c->phase != PH_DONE && s_ctl.err == 0) ? 1 : 0;
                if (go && step >= max_steps) {
                    s_ctl.err |= ERR_LEVEL_CAP;
                    go = 0;
                }
                s_go = go;
            }
            __syncthreads();
            if (!s_go) break;
            batch_step_body<MODE, NW, true>(LdsArgs{&s_a}, &s_ctl, 0, 0u, 1u);
        }
    }
    // state and statistics back for the host
    __syncthreads();
    SoloState &g = ra.states[blockIdx.x];
    for (int i = tid; i < (int)(sizeof(Head) / 8); i += NT)
        ((unsigned long long *)&g.h)[i] = ((const unsigned long long *)c)[i];
    if (tid == 0) g.err = s_ctl.err;
    for (int i = tid; i < kSoloLevels * 8; i += NT) {
        const unsigned long long x = ((const unsigned long long *)s_ctl.lvl)[i];
        if (x) (void)atomicAdd((unsigned long long *)ra.a.lvl + i, x);
    }
}

template __global__ void block_run<0, kBlockWaves>(BlockArgs);

}  // namespace bcx
