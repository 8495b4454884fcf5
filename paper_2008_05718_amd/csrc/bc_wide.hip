// bc_wide.hip -- Brandes on graphs with positive integer arc weights, up to 64
// sources traversed together by the whole GPU.
//
// Same phases as the engines that give a batch to one workgroup
// (bc_wbatch.hip, bc_weighted.hip), following the paper's forward "BFS
// traversal or SSSP calculation" and its dependency sweep (Section
// "Background", Eq. 2), as steps of a device-resident state machine like the
// unweighted batched engine (bc_batched.hip): one launch per round, the last
// workgroup moves the machine on.
//   WP_RELAX  one relaxation round: every queued vertex v (lanes m: the sources
//             whose distance to v dropped) offers dist + weight over its out-arcs;
//             a wavefront holds one arc's row of distances (lane = source),
//             lowers it by 64-bit atomicMin where the offer is smaller, and
//             marks those lanes of the far end for the next round.
//   WP_MARK   over every reached vertex once: for each out-arc the mask of the
//             lanes for which it lies on a shortest path, kept per arc in out-arc and in
//             in-arc order, and the in-arc counts of every (vertex, lane).
//             Few arcs are on a shortest path, so the phases below read 8 bytes per arc
//             instead of testing a row of distances per arc.
//   WP_DAG    one round of vertices whose predecessors are complete: path
//             counts summed over the marked in-arcs in CSR order (exact uint64 with
//             carries, or FP64 in mode 1), then the in-arc counts of the marked
//             successors go down, and those that reach zero form the next round.
//   WP_BWD    the rounds in reverse: delta = sigma * sum of c over the marked
//             out-arcs in CSR order.
//   WP_BC     scores in source order, reset of the distances.
//
// Against a batch per workgroup, a list of sources much shorter than 16 per
// compute unit still fills the GPU, the state is one batch's (0.15 GB instead of
// 12 GB at 65,536 vertices), and a vertex's arcs are read for 64 sources at
// a time.  Distances, marks and counts change by integer atomics, exact in any order;
// sums of doubles have an order fixed by the vertex.  Queue order changes no value.
//
// A relaxation round may read a distance that another workgroup lowers in
// the same round: distances only fall, so the offer is at most too large, and
// whoever lowered it has marked the vertex for the next round, which starts in
// a launch of its own and reads the new value.
#include "bc_common.h"

namespace bcx {
constexpr int kUnroll = 16;  // matched arcs whose rows are loaded together (R-MAT 2^16, 512 sources: 19.4 ms, 19.8 with 8)
}
#include "bc_rows.h"

namespace bcx {

namespace {

constexpr unsigned long long kInf = ~0ull;

struct WideScratch {
    Packing pk;
    Stage st;
};

struct RelaxCounters {
    unsigned long long arcs = 0, larcs = 0;
};

// Offers of the arcs of one chunk (lane j: arc j with far end x and weight w,
// `cnt` of them): per arc the row of the far end's distances against the
// entry's distance plus the weight.  ONE: all arcs belong to one entry (lanes
// m1, distances dv1); else lane own of the group holds the arc's entry
// (lanes M, row address er).  Returns, in lane j, the lanes for which the offer
// of arc j was smaller (RELAX; the far end's distance is lowered) or equal
// (MARK; the far end's in-arc count goes up).
template <bool MARK, bool ONE>
__device__ __forceinline__ unsigned long long offer_arcs(const WideArgs &a, int cnt, int x, int w, int own,
                                                         unsigned long long M, unsigned long long er,
                                                         unsigned long long m1, unsigned long long dv1) {
    constexpr int kT = 8;  // arcs whose rows are loaded together
    const int lane = lane_id();
    const unsigned long long xr = row_addr(a.dist, x, a.shift);
    unsigned long long hit = 0;
    for (int j = 0; j < cnt; j += kT) {
        unsigned long long dx[kT], dv[kT], mq[kT];
#pragma unroll
        for (int q = 0; q < kT; ++q) {
            const int jj = min(j + q, cnt - 1);
            const int o = ONE ? 0 : __builtin_amdgcn_readlane(own, jj);
            mq[q] = j + q < cnt ? (ONE ? m1 : readlane_u64(M, o)) : 0ull;
            const unsigned slot = row_slot(mq[q]);
            dx[q] = row_load(readlane_u64(xr, jj), slot);
            if (!ONE) dv[q] = row_load(readlane_u64(er, o), slot);
        }
#pragma unroll
        for (int q = 0; q < kT; ++q) {
            const int jj = min(j + q, cnt - 1);
            const unsigned long long nd =
                (ONE ? dv1 : dv[q]) + (unsigned long long)(unsigned)__builtin_amdgcn_readlane(w, jj);
            // lanes outside the mask loaded zero: no offer is below that
            const unsigned long long b = MARK ? (__ballot(nd == dx[q]) & mq[q]) : __ballot(nd < dx[q]);
            if (!b) continue;
            const int xj = __builtin_amdgcn_readlane(x, jj);
            if (__builtin_amdgcn_inverse_ballot_w64(b)) {
                const size_t at = ((size_t)(unsigned)xj << (a.shift - 3)) + lane;
                if (MARK) (void)atomicAdd(&a.cnt[at], 1);
                else (void)atomicMin(&a.dist[at], nd);
            }
            if (lane == jj) hit = b;
        }
    }
    return hit;
}

// Class degree of a vertex that joins a round.
struct WideDeg {
    const GraphArgs &g;
    __device__ __forceinline__ int operator()(int x, bool) const {
        return class_deg(g, x, g.row_ptr[x + 1] - g.row_ptr[x]);
    }
};

// Arcs that enter the next round's queue, or that are recorded (MARK).
struct NextRound {
    unsigned long long *mask;  // [n] marks of the next round
    StageTo<Ctl, WideDeg> to;
};

// Mark the lanes `hit` of x (per thread) for the next round; a vertex marked
// for the first time is queued.
__device__ __forceinline__ void mark_next(const WideArgs &a, const NextRound &nx, int x, unsigned long long hit,
                                          Stage &st, int &sn) {
    bool newly = false;
    if (hit) newly = atomicOr(&nx.mask[x], hit) == 0ull;
    stage_push(newly, x, st, sn, nx.to);
}

template <bool MARK>
__device__ __forceinline__ void offer_done(const WideArgs &a, const NextRound &nx, bool on, int e, int x,
                                           unsigned long long hit, Stage &st, int &sn) {
    if (MARK) {
        if (on) {
            a.dag_out[e] = hit;
            a.dag_in[a.rev[e]] = hit;
        }
    } else {
        mark_next(a, nx, x, on ? hit : 0ull, st, sn);
    }
}

// One entry's arcs [a0, a1) (uniform), lanes m, its distances dv.
template <bool MARK>
__device__ __forceinline__ void offer_entry(const WideArgs &a, const NextRound &nx, unsigned long long m,
                                            unsigned long long dv, int a0, int a1, Stage &st, int &sn,
                                            RelaxCounters &rc) {
    const int lane = lane_id();
    if (a0 >= a1) return;
    int x = a.g.col[min(a0 + lane, a1 - 1)], w = a.wt[min(a0 + lane, a1 - 1)];
    for (int eb = a0; eb < a1; eb += kWave) {
        const int cnt = min(kWave, a1 - eb), xc = x, wc = w;
        if (eb + kWave < a1) {
            x = a.g.col[min(eb + kWave + lane, a1 - 1)];
            w = a.wt[min(eb + kWave + lane, a1 - 1)];
        }
        const unsigned long long hit = offer_arcs<MARK, true>(a, cnt, xc, wc, 0, 0ull, 0ull, m, dv);
        offer_done<MARK>(a, nx, lane < cnt, eb + lane, xc, hit, st, sn);
    }
    if (lane == 0) {
        rc.arcs += (unsigned)(a1 - a0);
        rc.larcs += (unsigned long long)(unsigned)(a1 - a0) * (unsigned)__popcll(m);
    }
}

// The entries of one group: this lane's entry is vertex v with lanes M.
// Arcs of a vertex with no lanes are not followed, but where they can lead to a
// reached vertex (directed graphs) MARK records that they are on no shortest path.
template <bool MARK>
__device__ __forceinline__ void offer_group(const WideArgs &a, const NextRound &nx, bool valid, int v, unsigned long long M,
                                            WideScratch &ws, int &sn, RelaxCounters &rc) {
    const int lane = lane_id();
    const bool take = valid && (M != 0ull || (MARK && a.g.directed));
    const int e0 = take ? a.g.row_ptr[v] : 0;
    const int na = take ? a.g.row_ptr[v + 1] - e0 : 0;
    const int deg = take ? class_deg(a.g, v, na) : 0;
    const bool light = take && deg <= kPack, medium = take && deg > kPack && deg <= seg_arcs(a.g);
    const unsigned long long er = row_addr(a.dist, v, a.shift);
    int off;
    const int total = pack_entries(ws.pk, light ? na : 0,
                                   make_uint4((unsigned)e0, (unsigned)M, (unsigned)(M >> 32), (unsigned)lane),
                                   make_uint4(0u, 0u, 0u, 0u), off);
    if (total) {
        int before = 0;
        uint4 r = ws.pk.rec[packed_rank(ws.pk, 0, before)];
        int e = (int)r.x + min(lane, total - 1);
        int x = a.g.col[e], w = a.wt[e];
        unsigned larcs = 0;
        for (int base = 0; base < total; base += kWave) {
            const int cnt = min(kWave, total - base), xc = x, wc = w, ec = e, oc = (int)r.w;
            const bool on = lane < cnt;
            if (on) larcs += (unsigned)(__popc(r.y) + __popc(r.z));
            if (base + kWave < total) {
                r = ws.pk.rec[packed_rank(ws.pk, base / kWave + 1, before)];
                e = (int)r.x + min(base + kWave + lane, total - 1);
                x = a.g.col[e];
                w = a.wt[e];
            }
            const unsigned long long hit = offer_arcs<MARK, false>(a, cnt, xc, wc, oc, M, er, 0ull, 0ull);
            offer_done<MARK>(a, nx, on, ec, xc, hit, ws.st, sn);
        }
        rc.larcs += larcs;
        if (lane == 0) rc.arcs += (unsigned)total;
    }
    for (unsigned long long mm = __ballot(medium); mm; mm &= mm - 1) {
        const int j = __ffsll(mm) - 1;
        const int a0 = __builtin_amdgcn_readlane(e0, j);
        const unsigned long long mj = readlane_u64(M, j);
        const unsigned long long dv = row_load(readlane_u64(er, j), row_slot(mj));
        offer_entry<MARK>(a, nx, mj, dv, a0, a0 + __builtin_amdgcn_readlane(na, j), ws.st, sn, rc);
    }
    wave_lds_fence();  // the next group reuses the packing
}

// Release over one chunk of out-arcs (per thread: far end x, lanes xm for
// which the arc is on a shortest path from an entry of this round): the far
// end's in-arc counts go down; lanes that reach zero are ready.
__device__ __forceinline__ void release_chunk(const WideArgs &a, const NextRound &nx, int x, unsigned long long xm,
                                              Stage &st, int &sn) {
    const int lane = lane_id();
    unsigned long long ready = 0;
    for (unsigned long long bal = __ballot(xm != 0ull); bal;) {
        int old[4], jq[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            jq[q] = bal ? __ffsll(bal) - 1 : 0;
            const unsigned long long m = bal ? readlane_u64(xm, jq[q]) : 0ull;
            bal &= bal - 1;
            old[q] = 0;
            if (__builtin_amdgcn_inverse_ballot_w64(m))
                old[q] = atomicSub(
                    &a.cnt[((size_t)(unsigned)__builtin_amdgcn_readlane(x, jq[q]) << (a.shift - 3)) + lane], 1);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned long long b = __ballot(old[q] == 1);
            if (b && lane == jq[q]) ready = b;
        }
    }
    mark_next(a, nx, x, ready, st, sn);
}

__device__ __forceinline__ void release_entry(const WideArgs &a, const NextRound &nx, unsigned long long m, int a0,
                                              int a1, Stage &st, int &sn) {
    const int lane = lane_id();
    for (int eb = a0; eb < a1; eb += kWave) {
        const int e = min(eb + lane, a1 - 1);
        const unsigned long long xm = eb + lane < a1 ? (a.dag_out[e] & m) : 0ull;
        release_chunk(a, nx, a.g.col[e], xm, st, sn);
    }
}

// Path counts of a group's entries (rounds after the first) and release of
// their successors.
template <int MODE>
__device__ __forceinline__ void dag_group(const WideArgs &a, const NextRound &nx, const unsigned long long *mask, int l,
                                          int qb, int i0, int i1, WideScratch &ws, int &sn, unsigned long long &ovf,
                                          ArcCounters &ac) {
    constexpr int OP = MODE ? OP_F64 : OP_U64;
    const int lane = lane_id();
    const bool valid = i0 + lane < i1;
    const int p = qb + i0 + lane;
    const int v = valid ? a.lq_vtx[p] : 0;
    const unsigned long long M = valid ? mask[v] : 0ull;
    const int o0 = valid ? a.g.row_ptr[v] : 0, no = valid ? a.g.row_ptr[v + 1] - o0 : 0;
    const int n0 = (valid && a.g.directed) ? a.g.in_row_ptr[v] : o0;
    const int ni = (valid && a.g.directed) ? a.g.in_row_ptr[v + 1] - n0 : no;
    const int deg = max(no, ni);
    const bool light = valid && deg <= kPack, medium = valid && deg > kPack && deg <= seg_arcs(a.g);
    if (light || medium) a.lq_mask[p] = M;
    int off;
    if (l > 0) {
        const Slab sigma(a.sigma, a.shift);
        const unsigned long long ra = sigma.row(v);
        SigCounters sc;
        auto fin = [&](int e, const RowSum<OP> &s) {
            sig_store<OP>(s, readlane_u64(M, e), readlane_u64(ra, e), a.sigma_limit, ovf, sc);
        };
        const int total = pack_entries(ws.pk, light ? ni : 0,
                                       make_uint4((unsigned)n0, (unsigned)M, (unsigned)(M >> 32), (unsigned)lane),
                                       make_uint4(0u, 0u, 0u, 0u), off);
        RowSum<OP> acc;
        int cur;
        row_packed<OP>(ws.pk, total, ArcLanes{a.dag_in}, 0, a.g.in_col, sigma, acc, cur, ac, fin);
        if (cur >= 0) fin(cur, acc);
        for (unsigned long long mm = __ballot(medium); mm; mm &= mm - 1) {
            const int j = __ffsll(mm) - 1;
            const int a0 = __builtin_amdgcn_readlane(n0, j);
            RowSum<OP> sum;
            row_arcs<OP>(ArcLanes{a.dag_in}, readlane_u64(M, j), a0, a0 + __builtin_amdgcn_readlane(ni, j), 0,
                         a.g.in_col, sigma, sum, ac);
            fin(j, sum);
        }
        wave_lds_fence();
    }
    const int total = pack_entries(ws.pk, light ? no : 0,
                                   make_uint4((unsigned)o0, (unsigned)M, (unsigned)(M >> 32), (unsigned)lane),
                                   make_uint4(0u, 0u, 0u, 0u), off);
    int before = 0;
    for (int base = 0; base < total; base += kWave) {
        const uint4 r = ws.pk.rec[packed_rank(ws.pk, base / kWave, before)];
        const int e = (int)r.x + min(base + lane, total - 1);
        const unsigned long long xm =
            base + lane < total ? (a.dag_out[e] & (((unsigned long long)r.z << 32) | r.y)) : 0ull;
        release_chunk(a, nx, a.g.col[e], xm, ws.st, sn);
    }
    if (lane == 0) ac.arcs += (unsigned)total;
    for (unsigned long long mm = __ballot(medium); mm; mm &= mm - 1) {
        const int j = __ffsll(mm) - 1;
        const int a0 = __builtin_amdgcn_readlane(o0, j), nj = __builtin_amdgcn_readlane(no, j);
        release_entry(a, nx, readlane_u64(M, j), a0, a0 + nj, ws.st, sn);
        if (lane == 0) ac.arcs += (unsigned)nj;
    }
    wave_lds_fence();
}

template <int MODE>
__device__ __forceinline__ void back_group(const WideArgs &a, int qb, int i0, int i1, unsigned long long dead,
                                           WideScratch &ws, ArcCounters &ac) {
    const int lane = lane_id();
    const bool valid = i0 + lane < i1;
    const int p = qb + i0 + lane;
    const int v = valid ? a.lq_vtx[p] : 0;
    const int e0 = valid ? a.g.row_ptr[v] : 0, na = valid ? a.g.row_ptr[v + 1] - e0 : 0;
    const int deg = valid ? class_deg(a.g, v, na) : 0;
    const bool light = valid && deg <= kPack, medium = valid && deg > kPack && deg <= seg_arcs(a.g);
    const unsigned long long M = (light || medium) ? (a.lq_mask[p] & ~dead) : 0ull;
    const Slab sigma(a.sigma, a.shift), chat(a.chat, a.shift), delta(a.delta, a.shift);
    unsigned long long parked = 0;
    auto fin = [&](int e, const RowSum<OP_C> &s) {
        row_store(delta.row(__builtin_amdgcn_readlane(v, e)), row_slot(readlane_u64(M, e)), as_u64(s.d));
        parked |= 1ull << e;
    };
    int off, cur;
    const int total = pack_entries(ws.pk, (light && M) ? na : 0,
                                   make_uint4((unsigned)e0, (unsigned)M, (unsigned)(M >> 32), (unsigned)lane),
                                   make_uint4(0u, 0u, 0u, 0u), off);
    RowSum<OP_C> acc;
    row_packed<OP_C>(ws.pk, total, ArcLanes{a.dag_out}, 0, a.g.col, chat, acc, cur, ac, fin);
    if (cur >= 0) fin(cur, acc);
    for (unsigned long long mm = __ballot(medium && M != 0ull); mm; mm &= mm - 1) {
        const int j = __ffsll(mm) - 1;
        const int a0 = __builtin_amdgcn_readlane(e0, j);
        RowSum<OP_C> sum;
        row_arcs<OP_C>(ArcLanes{a.dag_out}, readlane_u64(M, j), a0, a0 + __builtin_amdgcn_readlane(na, j), 0, a.g.col,
                       chat, sum, ac);
        fin(j, sum);
    }
    bwd_finish<MODE>(__ballot(M != 0ull), parked, M, v, sigma, chat, delta, 0, 0);
    wave_lds_fence();
}

// Set up batch b (last workgroup, all threads): its sources are the first
// round of the relaxation and of the DAG rounds.
template <int MODE>
__device__ __forceinline__ void wide_begin(const WideArgs &a, Ctl *gc, Head *c, int64_t b, int *s_src, int *s_lead) {
    const int t = threadIdx.x;
    const int64_t start = a.batch_start[b];
    const int lanes = (int)(a.batch_start[b + 1] - start);
    if (t < kLanes) {
        const int s = t < lanes ? a.srcs[start + t] : -1;
        s_src[t] = s;
        a.lane_src[t] = s;
    }
    __syncthreads();
    if (t < lanes) {
        const int s = s_src[t];
        unsigned long long m = 0;
        int lead = t;
        for (int k = lanes - 1; k >= 0; --k)
            if (s_src[k] == s) {
                m |= 1ull << k;
                lead = k;
            }
        s_lead[t] = lead;
        const size_t at = ((size_t)(unsigned)s << (a.shift - 3)) + t;
        a.dist[at] = 0ull;
        a.sigma[at] = MODE ? as_u64(1.0) : 1ull;
        if (lead == t) {
            a.fm[s] = m;
            a.rdy[s] = m;
        }
    }
    __syncthreads();
    if (t == 0) {
        uint32_t cnt = 0, cost = 0;
        int nh = 0, segs = 0;
        for (int k = 0; k < lanes; ++k) {
            if (s_lead[k] != k) continue;  // lanes with the same source share an entry
            const int s = s_src[k];
            const int deg = class_deg(a.g, s, a.g.row_ptr[s + 1] - a.g.row_ptr[s]);
            a.rq[cnt] = s;
            a.lq_vtx[cnt] = s;
            const uint32_t ce = entry_cost(deg, a.g.seg_log);
            for (uint32_t g = cost / kBudget + 1; g <= (cost + ce) / kBudget; ++g) {
                a.rgs[g] = cnt + 1u;
                a.gstart[g] = cnt + 1u;
            }
            cost += ce;
            if (deg > seg_arcs(a.g)) {
                a.rhq.pos[nh] = (int32_t)cnt;
                a.rhq.seg[nh] = segs;
                a.hq.pos[nh] = (int32_t)cnt;
                a.hq.seg[nh] = segs;
                a.hq.cnt[nh] = 0;
                segs += n_segments(a.g, deg);
                ++nh;
            }
            ++cnt;
        }
        const uint32_t ng = (cost - 1u) / (uint32_t)kBudget + 1u;
        a.rgs[0] = 0u;
        a.rgs[ng] = cnt;
        a.gstart[0] = 0u;
        a.gstart[ng] = cnt;
        a.gbase[0] = 0u;
        a.gbase[1] = ng + 1u;
        a.hq.off[0] = 0;
        a.hq.off[1] = nh;
        a.hq.nseg[0] = segs;
        a.level_off[0] = 0;
        a.level_off[1] = (int32_t)cnt;
        c->w_cnt = cnt;
        c->w_groups = ng;
        c->w_heavy = nh;
        c->w_hsegs = segs;
        gc->next_qc = 0ull;
        gc->next_hq = 0ull;
        c->visited_n = 0ull;  // no round before
        c->pos = b;
        c->lanes = lanes;
        c->lane_mask = lanes >= 64 ? ~0ull : ((1ull << lanes) - 1ull);
        c->dead = 0ull;
        c->level = 0;
        c->n_levels = 0;
        const int64_t dp = c->dump_pos;
        c->dump_lane = (dp >= start && dp < start + lanes && c->dump_state == 0) ? (int)(dp - start) : -1;
        c->st_batches += 1;
        c->phase = WP_RELAX;
    }
}

}  // namespace

template <int MODE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void wide_step(WideArgs a) {
    constexpr int OP = MODE ? OP_F64 : OP_U64;
    __shared__ int s_phase, s_level, s_last, s_qb, s_qe, s_dlane, s_cnt, s_h0, s_h1, s_hseg, s_prev0, s_prev1;
    __shared__ uint32_t s_gb, s_ng;
    __shared__ unsigned s_nblk;
    __shared__ unsigned long long s_dead, s_lmask;
    __shared__ unsigned long long s_red[kWavesPerBlock * kNCnt];
    __shared__ Head s_head;
    __shared__ unsigned long long s_tot[kNCnt];
    __shared__ int s_src[kLanes], s_lead[kLanes];
    __shared__ StageTotals<kWavesPerBlock> s_stot;
    __shared__ union {
        WideScratch ws;
        double tile[kWave * 8];
    } s_scratch[kWavesPerBlock];
    Ctl *gc = a.ctl;
    Head *c = &s_head;
    head_load<kBlock>(s_head, gc->h[a.parity]);
    const int tid = threadIdx.x, lane = tid & 63, wid = uniform(tid >> 6);
    const unsigned bid = blockIdx.x, grid = gridDim.x;
    const int n = a.g.n;
    __syncthreads();
    if (tid == 0) {
        const int ph = c->phase, l = c->level;
        s_phase = ph;
        s_level = l;
        s_dead = c->dead;
        s_lmask = c->lane_mask;
        s_dlane = c->dump_lane;
        s_qb = s_qe = s_h0 = s_h1 = s_hseg = 0;
        s_gb = s_ng = 0;
        s_prev0 = s_prev1 = 0;  // entries of the round before, whose masks are cleared
        long long items = 1;
        if (ph == WP_RELAX) {
            const int r = l % 3;
            s_qb = r * n;
            s_qe = r * n + (int)c->w_cnt;
            s_gb = (uint32_t)r * a.rgcap;
            s_ng = c->w_groups;
            s_h0 = r * (int)a.rhcap;
            s_h1 = s_h0 + c->w_heavy;
            s_hseg = c->w_hsegs;
            s_prev1 = (int)c->visited_n;  // entries of round l - 1
        } else if (ph == WP_MARK) {
            s_ng = (uint32_t)a.n_sgroups;
            s_hseg = a.g.hv_seg[a.g.n_heavy];
            s_h1 = a.g.n_heavy;
            s_prev1 = (int)c->visited_n;  // entries of the last round (number l)
        } else if (ph == WP_DAG || ph == WP_BWD) {
            s_qb = a.level_off[l];
            s_qe = a.level_off[l + 1];
            s_gb = a.gbase[l];
            s_ng = a.gbase[l + 1] - s_gb - 1u;
            s_h0 = a.hq.off[l];
            s_h1 = a.hq.off[l + 1];
            s_hseg = a.hq.nseg[l];
            if (ph == WP_DAG && l > 0) {
                s_prev0 = a.level_off[l - 1];
                s_prev1 = s_qb;
            }
        }
        if (ph == WP_RELAX || ph == WP_MARK || ph == WP_DAG || ph == WP_BWD)
            items = (long long)s_ng + s_hseg + (s_prev1 - s_prev0) / (8 * kWave);
        else if (ph == WP_BC) items = (n + kWave - 1) / kWave;
        else if (ph == WP_DUMP) items = (n + kWave - 1) / kWave;
        s_nblk = active_blocks(items, grid);
    }
    __syncthreads();
    const int phase = uniform(s_phase);
    if (phase == PH_DONE || phase == PH_IDLE) return;
    const unsigned nblk = (unsigned)uniform((int)s_nblk);
    if (bid >= nblk) return;  // no work for this workgroup
    const int l = uniform(s_level);
    const int hseg = uniform(s_hseg), h0 = uniform(s_h0), h1 = uniform(s_h1);
    int n_groups = uniform((int)s_ng);
    const int ng = n_groups, gm = merge_groups((uint32_t)ng, grid * kWavesPerBlock);
    n_groups = (ng + gm - 1) / gm;  // consecutive groups of a large round are taken together
    const int total = n_groups + hseg;
    const int32_t *rp = a.g.row_ptr;
    WideScratch &ws = s_scratch[wid].ws;
    RelaxCounters rc;
    ArcCounters ac;
    unsigned long long ovf = 0, lent = 0;
    int sn = 0;
    if (phase == WP_RELAX || phase == WP_MARK) {
        const bool mark = phase == WP_MARK;
        const int r = l % 3, rn = (l + 1) % 3, rp3 = (l + 2) % 3;
        unsigned long long *fc = a.fm + (size_t)r * n;
        // clear the masks of the round before (of the last round when marking)
        {
            unsigned long long *fz = mark ? fc : a.fm + (size_t)rp3 * n;
            const int32_t *qz = a.rq + (size_t)(mark ? r : rp3) * n;
            const int cz = uniform(s_prev1);
            for (int i = (int)bid * kBlock + tid; i < cz; i += (int)nblk * kBlock) fz[qz[i]] = 0ull;
        }
        GroupArgs gr;
        gr.gstart = a.rgs;
        gr.gb = (uint32_t)rn * a.rgcap;
        gr.gcap = gr.gb + a.rgcap;
        const uint32_t qbase = (uint32_t)rn * (uint32_t)n;
        const NextRound nx{a.fm + (size_t)rn * n, stage_to(gc, a.rq, qbase, qbase + (uint32_t)n, a.rhq,
                                                           (uint32_t)rn * a.rhcap, gr, a.g, WideDeg{a.g})};
        const int qb = uniform(s_qb), cnt = mark ? n : uniform(s_qe) - qb;
        const uint32_t *gs = mark ? a.sgs : a.rgs + uniform((int)s_gb);
        const unsigned long long all = uniform(s_lmask);
        for (WorkCursor<> wc(gc, nblk, bid); wc.item() < total; wc.next(total)) {
            const int k = wc.item();
            const int it = k < hseg ? n_groups + k : k - hseg;  // heavy segments first
            if (it < n_groups) {
                const int i0 = uniform((int)gs[it * gm]), i1 = min(uniform((int)gs[min(it * gm + gm, ng)]), cnt);
                if (i1 <= i0) continue;
                const bool valid = i0 + lane < i1;
                if (!mark) {
                    const int v = valid ? a.rq[qb + i0 + lane] : 0;
                    const unsigned long long M = valid ? fc[v] : 0ull;
                    offer_group<false>(a, nx, valid, v, M, ws, sn, rc);
                } else {
                    // the lanes that reached each vertex: the rows are read once,
                    // one per step, the masks stay in the vertices' lanes
                    const int v = i0 + lane;
                    unsigned long long M = 0;
                    for (int j = 0; j < i1 - i0; j += 4) {
                        unsigned long long d[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            d[q] = row_load(row_addr(a.dist, min(i0 + j + q, i1 - 1), a.shift), row_slot(all));
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const unsigned long long b = __ballot(d[q] != kInf) & all;
                            if (j + q >= i1 - i0) break;
                            if (lane == j + q) M = b;
                        }
                    }
                    if (valid) {
                        a.rm[v] = M;
                        lent += (unsigned)__popcll(M);
                    }
                    offer_group<true>(a, nx, valid, v, M, ws, sn, rc);
                }
                continue;
            }
            const int t = it - n_groups;
            const int32_t *sp = mark ? a.g.hv_seg : a.rhq.seg;
            const int h = uniform(seg_owner(sp, h0, h1, t));
            const int v = uniform(mark ? a.g.hv_vtx[h] : a.rq[a.rhq.pos[h]]);
            const int a0 = uniform(rp[v]) + ((t - uniform(sp[h])) << a.g.seg_log);
            const int a1 = max(a0, min(uniform(rp[v + 1]), a0 + seg_arcs(a.g)));
            const unsigned long long dall = row_load(row_addr(a.dist, v, a.shift), row_slot(all));
            const unsigned long long m = mark ? (__ballot(dall != kInf) & all) : uniform(fc[v]);
            if (!m && !(mark && a.g.directed)) continue;
            if (mark) offer_entry<true>(a, nx, m, dall, a0, a1, ws.st, sn, rc);
            else offer_entry<false>(a, nx, m, dall, a0, a1, ws.st, sn, rc);
        }
        if (!mark)
            stage_finish<kWavesPerBlock>(ws.st, sn, s_stot, nx.to);
    } else if (phase == WP_DAG) {
        const int qb = uniform(s_qb), qe = uniform(s_qe), cnt = qe - qb;
        const unsigned long long *mask = a.rdy + (size_t)(l % 3) * n;
        {
            unsigned long long *fz = a.rdy + (size_t)((l + 2) % 3) * n;
            const int z0 = uniform(s_prev0), z1 = uniform(s_prev1);
            for (int i = z0 + (int)bid * kBlock + tid; i < z1; i += (int)nblk * kBlock) fz[a.lq_vtx[i]] = 0ull;
        }
        GroupArgs gr;
        gr.gstart = a.gstart;
        gr.gb = a.gbase[l + 1];
        gr.gcap = a.gcap;
        const NextRound nx{a.rdy + (size_t)((l + 1) % 3) * n, stage_to(gc, a.lq_vtx, (uint32_t)qe, a.lq_cap, a.hq,
                                                                       (uint32_t)h1, gr, a.g, WideDeg{a.g})};
        const uint32_t *gs = a.gstart + uniform((int)s_gb);
        for (WorkCursor<> wc(gc, nblk, bid); wc.item() < total; wc.next(total)) {
            const int k = wc.item();
            const int it = k < hseg ? n_groups + k : k - hseg;  // heavy segments first
            if (it < n_groups) {
                const int i0 = uniform((int)gs[it * gm]), i1 = min(uniform((int)gs[min(it * gm + gm, ng)]), cnt);
                if (i1 > i0) dag_group<MODE>(a, nx, mask, l, qb, i0, i1, ws, sn, ovf, ac);
                continue;
            }
            const int t = it - n_groups;
            const int h = uniform(seg_owner(a.hq.seg, h0, h1, t));
            const int s0 = uniform(a.hq.seg[h]), s = t - s0;
            const int p = uniform(a.hq.pos[h]);
            const int v = uniform(a.lq_vtx[p]);
            const unsigned long long m = uniform(mask[v]);
            if (s == 0 && lane == 0) a.lq_mask[p] = m;
            const int o0 = uniform(rp[v]), o1 = uniform(rp[v + 1]);
            const int r0 = o0 + (s << a.g.seg_log), r1 = max(r0, min(o1, r0 + seg_arcs(a.g)));
            release_entry(a, nx, m, r0, r1, ws.st, sn);
            if (lane == 0) ac.arcs += (unsigned)(r1 - r0);
            if (l == 0) continue;
            const int e0 = uniform(a.g.in_row_ptr[v]), e1 = uniform(a.g.in_row_ptr[v + 1]);
            const int a0 = e0 + (s << a.g.seg_log), a1 = max(a0, min(e1, a0 + seg_arcs(a.g)));
            RowSum<OP> sum;
            row_arcs<OP>(ArcLanes{a.dag_in}, m, a0, a1, 0, a.g.in_col, Slab(a.sigma, a.shift), sum, ac);
            const size_t slot = (size_t)(s0 + s) * kLanes + lane;
            part_store(&a.hq.part_lo[slot], MODE ? as_u64(sum.d) : sum.lo);
            if (MODE == 0) part_store(&a.hq.part_hi[slot], sum.hi);
            const int ns = n_segments(a.g, max(o1 - o0, e1 - e0));
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
            SigCounters sc;
            sig_store<OP>(sum, m, row_addr(a.sigma, v, a.shift), a.sigma_limit, ovf, sc);
        }
        stage_finish<kWavesPerBlock>(ws.st, sn, s_stot, nx.to);
    } else if (phase == WP_BWD) {
        const int qb = uniform(s_qb), cnt = uniform(s_qe) - qb;
        const unsigned long long dead = uniform(s_dead);
        const uint32_t *gs = a.gstart + uniform((int)s_gb);
        for (WorkCursor<> wc(gc, nblk, bid); wc.item() < total; wc.next(total)) {
            const int k = wc.item();
            const int it = k < hseg ? n_groups + k : k - hseg;
            if (it < n_groups) {
                const int i0 = uniform((int)gs[it * gm]), i1 = min(uniform((int)gs[min(it * gm + gm, ng)]), cnt);
                if (i1 > i0) back_group<MODE>(a, qb, i0, i1, dead, ws, ac);
                continue;
            }
            const int t = it - n_groups;
            const int h = uniform(seg_owner(a.hq.seg, h0, h1, t));
            const int s0 = uniform(a.hq.seg[h]), s = t - s0;
            const int p = uniform(a.hq.pos[h]);
            const int v = uniform(a.lq_vtx[p]);
            const unsigned long long M = uniform(a.lq_mask[p]) & ~dead;
            const int e0 = uniform(rp[v]), e1 = uniform(rp[v + 1]);
            const int a0 = e0 + (s << a.g.seg_log), a1 = max(a0, min(e1, a0 + seg_arcs(a.g)));
            RowSum<OP_C> sum;
            if (M) row_arcs<OP_C>(ArcLanes{a.dag_out}, M, a0, a1, 0, a.g.col, Slab(a.chat, a.shift), sum, ac);
            part_store(&a.hq.part_lo[(size_t)(s0 + s) * kLanes + lane], as_u64(sum.d));
            const int ns = n_segments(a.g, uniform(class_deg(a.g, v, e1 - e0)));
            if (!seg_arrive(&a.hq.cnt[h], ns)) continue;
            double acc = 0.0;
            for (int k2 = 0; k2 < ns; ++k2) acc += as_f64(part_load(&a.hq.part_lo[(size_t)(s0 + k2) * kLanes + lane]));
            if (lane == 0) a.hq.cnt[h] = 0;
            const unsigned slot = row_slot(M);
            double delta, cc;
            bwd_values<MODE>(row_load(row_addr(a.sigma, v, a.shift), slot), acc, 0, 0, delta, cc);
            row_store(row_addr(a.chat, v, a.shift), slot, as_u64(cc));
            row_store(row_addr(a.delta, v, a.shift), slot, as_u64(delta));
        }
    } else if (phase == WP_DUMP) {
        const int k = s_dlane;
        const int src = a.lane_src[k];
        for (int i = (int)bid * kBlock + tid; i < n; i += (int)nblk * kBlock) {
            const size_t at = ((size_t)(unsigned)i << (a.shift - 3)) + k;
            const unsigned long long d = a.dist[at];
            a.dump_d[i] = d == kInf ? -1 : (int64_t)d;
            a.dump_sig[i] = d == kInf ? 0ull : a.sigma[at];
            a.dump_delta[i] = (d == kInf || i == src) ? 0.0 : a.delta[at];
        }
    } else if (phase == WP_BC) {
        // dependencies -> scores in lane order (the run's source order), 64
        // vertices per wavefront, their delta rows 8 lanes at a time through
        // LDS; then distances back to infinite and the DAG marks to none
        if (tid < kLanes) s_src[tid] = a.lane_src[tid];
        __syncthreads();
        const unsigned long long all = uniform(s_lmask), keep = all & ~uniform(s_dead);
        double *tile = s_scratch[wid].tile;
        bool bad = false;
        for (int base = ((int)bid * kWavesPerBlock + wid) * kWave; base < n; base += (int)nblk * kBlock) {
            const int v = base + lane;
            const unsigned long long rmv = v < n ? a.rm[v] : 0ull, vis = rmv & keep;
            if (v < n) {
                a.rdy[v] = 0ull;
                a.rdy[(size_t)n + v] = 0ull;
                a.rdy[2 * (size_t)n + v] = 0ull;
            }
            unsigned long long any = __ballot(rmv != 0ull);
            if (!any) continue;
            double b = vis ? a.bc[v] : 0.0;
            for (int c8 = 0; c8 < kLanes / 8; ++c8) {
                const unsigned m8 = (unsigned)(vis >> (8 * c8)) & 0xFFu;
                if (!__ballot(m8 != 0u)) continue;
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const int vi = 8 * r + (lane >> 3), kk = lane & 7;
                    const unsigned mv = (unsigned)__shfl((int)m8, vi);
                    double d = 0.0;
                    if ((mv >> kk) & 1u) d = a.delta[((size_t)(unsigned)(base + vi) << (a.shift - 3)) + 8 * c8 + kk];
                    tile[vi * 8 + (kk ^ (vi & 7))] = d;
                }
                wave_lds_fence();
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (((m8 >> j) & 1u) && s_src[8 * c8 + j] != v) {
                        const double d = tile[lane * 8 + (j ^ (lane & 7))];
                        if (MODE == 1 && !isfinite(d)) bad = true;
                        b += d;
                    }
                }
                wave_lds_fence();
            }
            if (vis) a.bc[v] = b;
            const unsigned slot = row_slot(all);
            for (; any; any &= any - 1)
                row_store(row_addr(a.dist, base + __ffsll(any) - 1, a.shift), slot, kInf);
        }
        if (bad) atomicOr(&gc->err, ERR_SIGMA_RANGE);
    }

    Counters cn;
    cn.v[SC_ARCS] = rc.arcs + ac.arcs;
    cn.v[SC_LARCS] = rc.larcs + ac.larcs;
    cn.v[SC_PAIRS] = ac.pairs;
    cn.v[SC_OVF] = ovf;
    cn.v[SC_LENT] = lent;
    if (!step_epilogue<kWavesPerBlock>(gc, cn, s_red, s_tot, &s_last, bid, nblk)) return;

    // ---- the last workgroup advances the state machine
    if (tid == 0) {
        c->st_steps += 1;
        c->st_parcs[phase] += s_tot[SC_ARCS];
        c->st_plarcs[phase] += s_tot[SC_LARCS];
        c->st_ppairs[phase] += s_tot[SC_PAIRS];
        c->st_lane_entries += s_tot[SC_LENT];
        const unsigned long long now = wall_clock64(), prev = c->last_tick;
        c->st_ticks[phase] += prev ? now - prev : 0ull;
        c->last_tick = now;
        int action = 0;
        const unsigned long long qc = ld_agent(&gc->next_qc), nh = ld_agent(&gc->next_hq);
        const uint32_t cnt = (uint32_t)qc, cost = (uint32_t)(qc >> 32);
        if (phase == WP_RELAX) {
            c->st_fwd_levels += 1;
            gc->next_qc = 0ull;
            gc->next_hq = 0ull;
            c->visited_n = c->w_cnt;  // the queue whose masks the next step clears
            if (cnt == 0) {
                c->phase = WP_MARK;
            } else if (l > n + 2) {  // cannot happen with positive weights
                gc->err |= ERR_LEVEL_CAP;
                c->phase = PH_DONE;
            } else {
                const uint32_t gb = (uint32_t)((l + 1) % 3) * a.rgcap, ng = (cost - 1u) / (uint32_t)kBudget + 1u;
                a.rgs[gb] = 0u;
                a.rgs[gb + ng] = cnt;
                c->w_cnt = cnt;
                c->w_groups = ng;
                c->w_heavy = (int)(uint32_t)nh;
                c->w_hsegs = (int)(nh >> 32);
                c->level = l + 1;
            }
        } else if (phase == WP_MARK) {
            c->level = 0;
            c->phase = WP_DAG;
        } else if (phase == WP_DAG) {
            c->st_var[0] += 1;
            gc->next_qc = 0ull;
            gc->next_hq = 0ull;
            const unsigned long long o = s_tot[SC_OVF] & ~c->dead;
            const int64_t start = a.batch_start[c->pos];
            for (unsigned long long x = o; x; x &= x - 1) {
                const uint32_t q = c->n_ovf;
                if (q < a.ovf_cap) a.ovf_list[q] = start + __ffsll(x) - 1;
                else gc->err |= ERR_OVF_CAP;
                c->n_ovf = q + 1;
            }
            c->dead |= o;
            if (cnt == 0) {
                const int L = l + 1;
                c->n_levels = L;
                if ((unsigned long long)L > c->st_max_levels) c->st_max_levels = L;
                if (L >= 2) {
                    c->level = L - 1;
                    c->phase = WP_BWD;
                } else {
                    action = 1;
                }
            } else if (l + 2 >= a.max_levels + 2) {
                gc->err |= ERR_LEVEL_CAP;
                c->phase = PH_DONE;
            } else {
                const uint32_t gb = s_gb + s_ng + 1u, ng = (cost - 1u) / (uint32_t)kBudget + 1u;
                if ((unsigned long long)gb + ng + 1u > a.gcap) {
                    gc->err |= ERR_QUEUE_CAP;
                    c->phase = PH_DONE;
                } else {
                    a.level_off[l + 2] = s_qe + (int)cnt;
                    a.gstart[gb] = 0u;
                    a.gstart[gb + ng] = cnt;
                    a.gbase[l + 2] = gb + ng + 1u;
                    a.hq.off[l + 2] = s_h1 + (int)(uint32_t)nh;
                    a.hq.nseg[l + 1] = (int)(nh >> 32);
                    c->level = l + 1;
                }
            }
        } else if (phase == WP_BWD) {
            if (l - 1 >= 1) c->level = l - 1;
            else action = 1;
        } else if (phase == WP_DUMP) {
            c->dump_state = 2;
            c->phase = WP_BC;
        } else if (phase == WP_BC) {
            const int64_t next = c->pos + 1;
            c->pos = next;
            c->phase = next < c->n_items ? WP_BEGIN : PH_DONE;
        }
        if (action == 1)  // the batch's sums are complete
            c->phase = (c->dump_lane >= 0 && !((c->dead >> c->dump_lane) & 1ull)) ? WP_DUMP : WP_BC;
        s_cnt = phase == WP_BEGIN;
    }
    __syncthreads();
    if (s_cnt) wide_begin<MODE>(a, gc, c, c->pos, s_src, s_lead);
    head_store(gc, s_head, a.parity);
}

template __global__ void wide_step<0>(WideArgs);
template __global__ void wide_step<1>(WideArgs);

}  // namespace bcx
