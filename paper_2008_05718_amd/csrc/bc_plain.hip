// bc_plain.hip -- plain Brandes engine: one source at a time, the whole GPU
// working on each BFS level (paper, Section "Background": the level loop of
// the algorithm figure "Betweenness Centrality Algorithm", parallelised over
// the frontier's vertices and edges as that section describes).
//
// One kernel, plain_step<MODE>, executes the current phase of a device-side
// state machine (forward discover / path counts / backward / reset).  The
// last workgroup of each launch advances the machine, so a run is a stream of
// identical launches that the host can capture in a hipGraph.
//
// MODE 0: path counts in uint64.  Push levels add sigma with 64-bit atomics
//         (order-independent, exact); the atomic that carries past 2^64 - 1
//         (or the test limit) flags the source, which is then skipped and
//         redone in MODE 1.
// MODE 1: path counts in FP64, scaled by one power of two per level:
//         sigma(v) = raw(v) * 2^(E_l), E_l = shift_0 + ... + shift_l.  Counts
//         are pulled in CSR order after discovery, so every summation order
//         is fixed by the vertex alone.
//
// Backward (both modes): delta(v) = sigma(v) * sum over successors w of
// c(w), c(w) = (1 + delta(w)) / sigma(w) -- Eq. 2 with sigma(v) factored
// out.  Each vertex's sum is formed by kSub lanes (degree <= kSubDeg), one
// wavefront (a segment) or segments combined in segment order by the
// last segment to finish; no floating-point atomics, so results are bitwise
// reproducible.
//
// What bounds a step is the chain of dependent loads behind an arc (vertex,
// row bounds, column, level, value), not bytes, so the arcs are spread over
// lanes and every lane requests kArcs of them together.  With a thread per
// vertex instead, up to 32 arcs after one another, 32 sources on R-MAT 18 took
// 27.3 ms and 4 on a damaged 512 x 512 grid 38.6; with this 13.5 and 24.5, and 10.9
// and 21.4 with four workgroups per compute unit and no word that all of them update.
#include "bc_common.h"

namespace bcx {

template <int MODE>
__device__ __forceinline__ double norm_sigma(const PlainArgs &a, int v, int sh) {
    if (MODE == 0) return (double)a.sig[v];
    return ldexp(as_f64(a.sig[v]), -sh);
}

// A vertex's arcs [e0, e0 + len) are worked on by a group of G consecutive
// lanes (kSub, or the wavefront), kArcs per lane at a time.
// (R-MAT 18, 32 sources, when a run took 13.5 ms: 8 lanes 13.5, 4 13.8, 16 14.2;
// 2, 4 and 8 arcs per lane 14.5, 13.5 and 14.0; up to 32, 64 and 128 arcs 13.7,
// 13.5 and 13.5.)
constexpr int kSub = 8;
constexpr int kSubDeg = 64;
constexpr int kArcs = 4;
constexpr int kPullRun = 4;
constexpr int kPullSpan = 32;  // vertices a wavefront looks over for unvisited ones
template <int G>
__device__ __forceinline__ bool group_any(bool x) {
    const unsigned long long b = __ballot(x);
    return G == kWave ? b != 0ull : ((b >> (lane_id() & ~(G - 1))) & ((1ull << (G & 63)) - 1)) != 0ull;
}

// Top-down over the arcs of a frontier vertex (path count sv): claim unvisited
// neighbours, add sv to the neighbours on level l+1 (MODE 0).
template <int MODE, int G, class To>
__device__ __forceinline__ void plain_push_arcs(const PlainArgs &a, int l, unsigned long long sv, int e0, int len,
                                                unsigned long long &my_larcs, int &my_ovf, Stage &st, int &sn,
                                                const To &to) {
    const int32_t *__restrict__ col = a.g.col;
    for (int t = lane_id() & (G - 1); __any(t < len); t += kArcs * G) {
        int w[kArcs], dv[kArcs];
        bool newly[kArcs];
#pragma unroll
        for (int q = 0; q < kArcs; ++q) w[q] = t + q * G < len ? col[e0 + t + q * G] : -1;
#pragma unroll
        for (int q = 0; q < kArcs; ++q) dv[q] = w[q] >= 0 ? a.d[w[q]] : -2;
#pragma unroll
        for (int q = 0; q < kArcs; ++q) {
            newly[q] = false;
            if (dv[q] == -1) {
                const int old = atomicCAS(&a.d[w[q]], -1, l + 1);
                newly[q] = (old == -1);
                dv[q] = newly[q] ? l + 1 : old;
            }
        }
#pragma unroll
        for (int q = 0; q < kArcs; ++q) {
            if (MODE == 0 && dv[q] == l + 1) {
                const unsigned long long old = atomicAdd(&a.sig[w[q]], sv);
                const unsigned long long nv = old + sv;
                if (nv < old || nv > a.sigma_limit) my_ovf = 1;
                ++my_larcs;
            }
        }
#pragma unroll
        for (int q = 0; q < kArcs; ++q) stage_push(newly[q], w[q], st, sn, to);
    }
}

// Bottom-up over the arcs of an unvisited vertex: is a neighbour on level l,
// and (MODE 0) the exact sum of such neighbours' path counts.  MODE 1 stops at
// the first round with one.  Every lane of the group gets the result.
template <int MODE, int G>
__device__ __forceinline__ bool plain_pull_arcs(const PlainArgs &a, int l, int e0, int len, unsigned long long &lo,
                                                unsigned long long &hi, unsigned long long &my_arcs,
                                                unsigned long long &my_larcs) {
    const int32_t *__restrict__ col = a.g.col;
    bool found = false;
    lo = 0;
    hi = 0;
    for (int t = lane_id() & (G - 1); __any(t < len && !(MODE == 1 && found)); t += kArcs * G) {
        int u[kArcs], du[kArcs];
        unsigned long long x[kArcs];
#pragma unroll
        for (int q = 0; q < kArcs; ++q)
            u[q] = t + q * G < len && !(MODE == 1 && found) ? col[e0 + t + q * G] : -1;
#pragma unroll
        for (int q = 0; q < kArcs; ++q) du[q] = u[q] >= 0 ? a.d[u[q]] : -2;
#pragma unroll
        for (int q = 0; q < kArcs; ++q) {
            my_arcs += u[q] >= 0 ? 1u : 0u;
            x[q] = MODE == 0 && du[q] == l ? a.sig[u[q]] : 0ull;
        }
        bool f = false;
#pragma unroll
        for (int q = 0; q < kArcs; ++q) {
            f |= du[q] == l;
            if (MODE == 0) {
                lo += x[q];
                hi += (lo < x[q]) ? 1ull : 0ull;
                my_larcs += du[q] == l ? 1u : 0u;
            }
        }
        if (MODE == 1) f = group_any<G>(f);
        found |= f;
    }
    if (MODE == 0) {
        found = group_any<G>(found);
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) {
            const unsigned long long ol = shfl_u64(lo, lane_id() ^ o), oh = shfl_u64(hi, lane_id() ^ o);
            const unsigned long long nl = lo + ol;
            hi = hi + oh + ((nl < lo) ? 1ull : 0ull);
            lo = nl;
        }
    }
    return found;
}

// Sum over a vertex's arcs of the values of neighbours u with d[u] == want:
// sigma (normalised by 2^-sh, MODE 1) or c.  Lane-strided, then a fixed
// butterfly: every lane of the group returns the same bits.
template <int G>
__device__ __forceinline__ double plain_sum(const PlainArgs &a, int e0, int len, int want, bool use_chat, int sh,
                                            unsigned long long &my_larcs) {
    const int32_t *__restrict__ col = a.g.col;
    double p = 0.0;
    for (int t = lane_id() & (G - 1); __any(t < len); t += kArcs * G) {
        int u[kArcs], du[kArcs];
        double x[kArcs];
#pragma unroll
        for (int q = 0; q < kArcs; ++q) u[q] = t + q * G < len ? col[e0 + t + q * G] : -1;
#pragma unroll
        for (int q = 0; q < kArcs; ++q) du[q] = u[q] >= 0 ? a.d[u[q]] : -2;
#pragma unroll
        for (int q = 0; q < kArcs; ++q) {
            x[q] = 0.0;
            if (du[q] == want) {
                x[q] = use_chat ? a.chat[u[q]] : as_f64(a.sig[u[q]]);
                ++my_larcs;
            }
        }
#pragma unroll
        for (int q = 0; q < kArcs; ++q) p += use_chat ? x[q] : ldexp(x[q], -sh);
    }
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) p += __shfl_xor(p, o);
    return p;
}

// Transition helpers run by the last workgroup (all threads present).
template <int MODE>
__device__ __forceinline__ void plain_begin_source(const PlainArgs &a, Ctl *gc, Head *c, int64_t pos, float *lds, LevelFeatures *sf) {
    if (threadIdx.x == 0) {
        const int s = a.srcs[pos];
        a.d[s] = 0;
        a.sig[s] = MODE ? as_u64(1.0) : 1ull;
        a.queue[0] = s;
        a.level_off[0] = 0;
        a.level_off[1] = 1;
        a.shift[0] = 0;
        const int deg = a.g.row_ptr[s + 1] - a.g.row_ptr[s];
        a.hq.off[0] = 0;
        if (deg > seg_arcs(a.g)) {  // heavy source: its level-0 push runs as segments
            a.hq.pos[0] = 0;
            a.hq.seg[0] = 0;
            a.hq.cnt[0] = 0;
            a.hq.off[1] = 1;
            a.hq.nseg[0] = n_segments(a.g, deg);
        } else {
            a.hq.off[1] = 0;
            a.hq.nseg[0] = 0;
        }
        gc->next_hq = 0;
        c->pos = pos;
        c->level = 0;
        gc->next_qc = 0ull;
        c->visited_n = 1;
        c->visited_m = (unsigned long long)deg;
        c->prev_variant = V_PUSH_TPV;
        c->phase = PH_FWD;
        (void)atomicAdd(&level_rec(a.lvl, 0).entries, 1ull);
        c->st_lane_entries += 1;
        sf->nf = 1.0f;
        sf->mf = (float)deg;
        sf->nu = (float)(a.g.n - 1);
        sf->mu = (float)((long long)a.g.nnz_lo - deg);
        sf->level = 0;
    }
    __syncthreads();
    int lbo;  // one source per entry: no summation options here
    const int v = choose_variant(a.p, c->policy, V_PUSH_TPV, *sf, (float)a.g.n, (float)a.g.nnz_lo, lds, &lbo);
    if (threadIdx.x == 0) c->variant = v;
}

template <int MODE>
__device__ __forceinline__ void plain_advance_level(const PlainArgs &a, Ctl *gc, Head *c, int l, uint32_t cnt, unsigned long long edges,
                                    float *lds, LevelFeatures *sf) {
    if (threadIdx.x == 0) {
        c->level = l + 1;
        c->visited_n += cnt;
        c->visited_m += edges;
        sf->nf = (float)cnt;
        sf->mf = (float)edges;
        sf->nu = (float)((long long)a.g.n - (long long)c->visited_n);
        sf->mu = (float)((long long)a.g.nnz_lo - (long long)c->visited_m);
        sf->level = l + 1;
        gc->next_qc = 0ull;
        c->prev_variant = c->variant;
        c->phase = PH_FWD;
    }
    __syncthreads();
    int lbo;
    const int v = choose_variant(a.p, c->policy, c->prev_variant, *sf, (float)a.g.n, (float)a.g.nnz_lo, lds, &lbo);
    if (threadIdx.x == 0) c->variant = v;
}

// After the forward of the current source ended with L levels.
__device__ __forceinline__ void plain_after_forward(const PlainArgs &a, Head *c, int L) {
    c->n_levels = L;
    if ((unsigned long long)L > c->st_max_levels) c->st_max_levels = L;
    if (c->dump_pos == c->pos && c->dump_state == 0) {
        c->phase = PH_DUMP_FWD;
    } else if (L >= 2) {
        c->phase = PH_BWD;
        c->level = L - 1;
    } else {
        c->phase = PH_FIN;
    }
}

template <int MODE>
__global__ __launch_bounds__(kBlock) void plain_step(PlainArgs a) {
    __shared__ int s_phase, s_level, s_variant, s_last, s_qb, s_qe, s_qn, s_sh0, s_sh1, s_dump;
    __shared__ int s_h0, s_h1, s_hseg, s_hqb;
    __shared__ unsigned s_nblk;
    __shared__ unsigned long long s_red[kWavesPerBlock * kNCnt];
    __shared__ Head s_head;
    __shared__ unsigned long long s_tot[kNCnt];
    __shared__ Stage s_stage[kWavesPerBlock];
    __shared__ StageTotals<kWavesPerBlock> s_stot;
    __shared__ float s_lds[2 * kMlpH + kMlpOut + 4];
    __shared__ LevelFeatures s_feat;
    Ctl *gc = a.ctl;
    Head *c = &s_head;
    head_load<kBlock>(s_head, gc->h[a.parity]);
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    __syncthreads();
    if (tid == 0) {
        s_phase = c->phase;
        s_level = c->level;
        s_variant = c->variant;
        s_dump = (c->dump_pos == c->pos && c->dump_state == 1) ? 1 : 0;
        const int l = s_level;
        s_qb = s_qe = s_qn = s_sh0 = s_sh1 = 0;
        s_h0 = s_h1 = s_hseg = s_hqb = 0;
        if (s_phase == PH_FWD || s_phase == PH_SIG || s_phase == PH_BWD) {
            s_qb = a.level_off[l];
            s_qe = a.level_off[l + 1];
            s_qn = (s_phase == PH_SIG) ? a.level_off[l + 2] : 0;
            s_sh0 = MODE ? a.shift[l] : 0;
            s_sh1 = (MODE && s_phase == PH_BWD && l + 1 < c->n_levels) ? a.shift[l + 1] : 0;
        } else if (s_phase == PH_FIN) {
            s_qe = (int)c->total_queued;
            // the next source's words are left to the last workgroup, which
            // sets them: a word stored by two workgroups of one launch ends
            // with whichever L2 writes it back last
            s_sh0 = c->pos + 1 < c->n_items ? a.srcs[c->pos + 1] : -1;
        }
        if (s_phase == PH_FWD) {
            if (s_variant == V_PULL) {  // static heavy vertices
                s_h0 = 0;
                s_h1 = a.g.n_heavy;
                s_hseg = a.g.hv_seg[a.g.n_heavy];
            } else {                    // heavy frontier vertices of level l
                s_h0 = a.hq.off[l];
                s_h1 = a.hq.off[l + 1];
                s_hseg = a.hq.nseg[l];
            }
            s_hqb = a.hq.off[l + 1];
        } else if (s_phase == PH_SIG) {
            s_h0 = a.hq.off[l + 1];
            s_h1 = a.hq.off[l + 2];
            s_hseg = a.hq.nseg[l + 1];
        } else if (s_phase == PH_BWD) {
            s_h0 = a.hq.off[l];
            s_h1 = a.hq.off[l + 1];
            s_hseg = a.hq.nseg[l];
        }
        // wavefront work items of this step -> workgroups taking part
        long long items = 1;
        const int cnt = s_qe - s_qb;
        if (s_phase == PH_FWD) {
            if (s_variant == V_PUSH_TPV) items = (cnt + kWave / kSub - 1) / (kWave / kSub) + s_hseg;
            else if (s_variant == V_PUSH_WPV) items = cnt + s_hseg;
            else items = (a.g.n + kPullSpan - 1) / kPullSpan + s_hseg;
        } else if (s_phase == PH_SIG) {
            items = (s_qn - s_qe + kWave / kSub - 1) / (kWave / kSub) + s_hseg;
        } else if (s_phase == PH_BWD) {
            items = (cnt + kWave / kSub - 1) / (kWave / kSub) + s_hseg;
        } else if (s_phase == PH_FIN) {
            items = (s_qe + kWave - 1) / kWave;
        } else if (s_phase == PH_DUMP_FWD) {
            items = (a.g.n + kWave - 1) / kWave;
        }
        s_nblk = active_blocks(items, gridDim.x);
    }
    __syncthreads();
    const int phase = s_phase;
    if (phase == PH_DONE || phase == PH_IDLE) return;
    const unsigned nblk = s_nblk;
    if (blockIdx.x >= nblk) return;  // no work for this workgroup

    const int gw = blockIdx.x * kWavesPerBlock + wid;
    const int nw = (int)nblk * kWavesPerBlock;
    const int l = s_level;
    const int n = a.g.n;
    const int32_t *__restrict__ rp = a.g.row_ptr;
    int32_t *d = a.d;
    unsigned long long *sig = a.sig;
    const int h0 = s_h0, h1 = s_h1, hseg = s_hseg;
    const int sub = lane / kSub;             // the lane's entry of a wavefront's kPer
    const bool lead = lane % kSub == 0;
    constexpr int kPer = kWave / kSub;

    unsigned long long my_edges = 0, my_arcs = 0, my_larcs = 0;
    int my_ovf = 0, my_maxe = INT_MIN, my_mine = INT_MAX;

    if (phase == PH_FWD) {
        const int qb = s_qb, qe = s_qe, cnt = qe - qb;
        const int variant = s_variant;
        const uint32_t hqb = (uint32_t)s_hqb;
        Stage &st = s_stage[wid];
        int sn = 0;
        const auto to = stage_to(gc, a.queue, (uint32_t)qe, (uint32_t)n, a.hq, hqb, GroupArgs{}, a.g,
                                 [&](int w, bool first) {
                                     const int deg = rp[w + 1] - rp[w];
                                     if (first) my_edges += (unsigned)deg;
                                     return deg;
                                 });
        if (variant == V_PUSH_TPV || variant == V_PUSH_WPV) {
            const int n_light = variant == V_PUSH_TPV ? (cnt + kPer - 1) / kPer : cnt;
            const int total = n_light + hseg;
            for (int k = gw; k < total; k += nw) {
                const int it = k < hseg ? n_light + k : k - hseg;  // heavy segments first
                if (it >= n_light) {  // a segment of a heavy frontier vertex
                    const int t = it - n_light;
                    const int h = seg_owner(a.hq.seg, h0, h1, t);
                    const int s = t - a.hq.seg[h];
                    const int v = a.queue[a.hq.pos[h]];
                    const int a0 = seg_begin(a.g, rp[v], s), a1 = seg_end(a.g, rp[v], rp[v + 1], s);
                    if (lane == 0) my_arcs += (unsigned)(a1 - a0);
                    const unsigned long long sv = MODE == 0 ? sig[v] : 0ull;
                    plain_push_arcs<MODE, kWave>(a, l, sv, a0, a1 - a0, my_larcs, my_ovf, st, sn, to);
                } else if (variant == V_PUSH_WPV) {
                    const int v = a.queue[qb + it];
                    const int e0 = rp[v], e1 = rp[v + 1];
                    if (e1 - e0 > seg_arcs(a.g)) continue;  // runs as segments
                    if (lane == 0) my_arcs += (unsigned)(e1 - e0);
                    const unsigned long long sv = MODE == 0 ? sig[v] : 0ull;
                    plain_push_arcs<MODE, kWave>(a, l, sv, e0, e1 - e0, my_larcs, my_ovf, st, sn, to);
                } else {  // TPV: kPer frontier vertices per wavefront
                    const int i = it * kPer + sub;
                    const bool valid = i < cnt;
                    const int v = valid ? a.queue[qb + i] : 0;
                    const int e0 = valid ? rp[v] : 0;
                    const int deg = valid ? rp[v + 1] - e0 : 0;
                    const unsigned long long sv = (MODE == 0 && valid) ? sig[v] : 0ull;
                    if (lead) my_arcs += (unsigned)(deg <= seg_arcs(a.g) ? deg : 0);
                    plain_push_arcs<MODE, kSub>(a, l, sv, e0, deg <= kSubDeg ? deg : 0, my_larcs,
                                                my_ovf, st, sn, to);
                    // medium-degree vertices: the whole wavefront, one at a time
                    unsigned long long mm = __ballot(lead && deg > kSubDeg && deg <= seg_arcs(a.g));
                    while (mm) {
                        const int j = __ffsll(mm) - 1;
                        mm &= mm - 1;
                        plain_push_arcs<MODE, kWave>(a, l, shfl_u64(sv, j), __shfl(e0, j), __shfl(deg, j),
                                                     my_larcs, my_ovf, st, sn, to);
                    }
                }
            }
        } else {  // V_PULL: every unvisited vertex looks for neighbours on level l
            const int n_light = (n + kPullSpan - 1) / kPullSpan;
            const int total = n_light + hseg;
            for (int k = gw; k < total; k += nw) {
                const int it = k < hseg ? n_light + k : k - hseg;  // heavy segments first
                if (it >= n_light) {  // a segment of a heavy vertex
                    const int t = it - n_light;
                    const int h = seg_owner(a.g.hv_seg, h0, h1, t);
                    const int s = t - a.g.hv_seg[h];
                    const int w = a.g.hv_vtx[h];
                    const int dw0 = d[w];
                    // unvisited before this level (another segment may have
                    // claimed it during this step)
                    if (dw0 != -1 && dw0 != l + 1) continue;
                    const int a0 = seg_begin(a.g, rp[w], s), a1 = seg_end(a.g, rp[w], rp[w + 1], s);
                    unsigned long long lo, hi;
                    const bool any = plain_pull_arcs<MODE, kWave>(a, l, a0, a1 - a0, lo, hi, my_arcs, my_larcs);
                    bool newly = false;
                    if (any) {
                        if (MODE == 0) {  // exact 128-bit sum of the segment, one atomic
                            if (lane == 0) {
                                const unsigned long long old = atomicAdd(&sig[w], lo);
                                const unsigned long long nv = old + lo;
                                if (hi != 0 || nv < old || nv > a.sigma_limit) my_ovf = 1;
                            }
                        }
                        if (lane == 0) newly = atomicCAS(&d[w], -1, l + 1) == -1;
                    }
                    stage_push(newly, w, st, sn, to);
                    continue;
                }
                // runs of kPullRun vertices from every part of the numbering: hubs
                // are numbered together, and a wavefront takes them one by one
                const int w0 = ((lane / kPullRun) * n_light + it) * kPullRun + lane % kPullRun;
                unsigned long long cm = __ballot(lane < kPullSpan && w0 < n && d[w0] == -1);
                while (cm) {  // kPer unvisited vertices at a time
                    int w = -1;
#pragma unroll
                    for (int j = 0; j < kPer; ++j) {
                        const int i = cm ? __ffsll(cm) - 1 : 0;
                        if (cm && sub == j) w = __builtin_amdgcn_readlane(w0, i);
                        cm &= cm - 1;
                    }
                    const int e0 = w >= 0 ? rp[w] : 0;
                    const int deg = w >= 0 ? rp[w + 1] - e0 : 0;
                    unsigned long long lo, hi;
                    bool found =
                        plain_pull_arcs<MODE, kSub>(a, l, e0, deg <= kSubDeg ? deg : 0, lo, hi, my_arcs, my_larcs);
                    // medium-degree candidates: the whole wavefront, one at a time
                    unsigned long long mm = __ballot(lead && deg > kSubDeg && deg <= seg_arcs(a.g));
                    while (mm) {
                        const int j = __ffsll(mm) - 1;
                        mm &= mm - 1;
                        unsigned long long ml, mh;
                        const bool mf = plain_pull_arcs<MODE, kWave>(a, l, __shfl(e0, j), __shfl(deg, j), ml, mh,
                                                                     my_arcs, my_larcs);
                        if (lane == j) {
                            found = mf;
                            lo = ml;
                            hi = mh;
                        }
                    }
                    const bool ok = lead && found && deg <= seg_arcs(a.g);
                    if (ok) {
                        d[w] = l + 1;
                        if (MODE == 0) {
                            sig[w] = lo;
                            if (hi != 0 || lo > a.sigma_limit) my_ovf = 1;
                        }
                    }
                    stage_push(ok, w, st, sn, to);
                }
            }
        }
        stage_finish<kWavesPerBlock>(st, sn, s_stot, to);
    } else if (MODE == 1 && phase == PH_SIG) {
        // FP64 path counts of level l+1, pulled in CSR order
        const int qs = s_qe, cnt = s_qn - s_qe;
        const int sh = s_sh0;
        const int n_light = (cnt + kPer - 1) / kPer;
        const int total = n_light + hseg;
        for (int k = gw; k < total; k += nw) {
            const int it = k < hseg ? n_light + k : k - hseg;  // heavy segments first
            if (it >= n_light) {  // a segment of a heavy new vertex
                const int t = it - n_light;
                const int h = seg_owner(a.hq.seg, h0, h1, t);
                const int s = t - a.hq.seg[h];
                const int w = a.queue[a.hq.pos[h]];
                const int e0 = rp[w], e1 = rp[w + 1];
                const int a0 = seg_begin(a.g, e0, s), a1 = seg_end(a.g, e0, e1, s);
                const double p = plain_sum<kWave>(a, a0, a1 - a0, l, false, sh, my_larcs);
                if (lane == 0) {
                    my_arcs += (unsigned)(a1 - a0);
                    part_store(&a.hq.part_lo[a.hq.seg[h] + s], as_u64(p));
                }
                const int ns = n_segments(a.g, e1 - e0);
                if (!seg_arrive(&a.hq.cnt[h], ns)) continue;
                if (lane == 0) {
                    double acc = 0.0;
                    for (int k = 0; k < ns; ++k) acc += as_f64(part_load(&a.hq.part_lo[a.hq.seg[h] + k]));
                    sig[w] = as_u64(acc);
                    if (acc > 0.0) {
                        int ex;
                        frexp(acc, &ex);
                        my_maxe = max(my_maxe, ex);
                        my_mine = min(my_mine, ex);
                    }
                    a.hq.cnt[h] = 0;
                }
                continue;
            }
            const int i = it * kPer + sub;
            const bool valid = i < cnt;
            const int w = valid ? a.queue[qs + i] : 0;
            const int e0 = valid ? rp[w] : 0;
            const int deg = valid ? rp[w + 1] - e0 : 0;
            if (lead) my_arcs += (unsigned)(deg <= seg_arcs(a.g) ? deg : 0);
            double acc = plain_sum<kSub>(a, e0, deg <= kSubDeg ? deg : 0, l, false, sh, my_larcs);
            unsigned long long mm = __ballot(lead && deg > kSubDeg && deg <= seg_arcs(a.g));
            while (mm) {
                const int j = __ffsll(mm) - 1;
                mm &= mm - 1;
                const double p = plain_sum<kWave>(a, __shfl(e0, j), __shfl(deg, j), l, false, sh, my_larcs);
                if (lane == j) acc = p;
            }
            if (lead && valid && deg <= seg_arcs(a.g)) {
                sig[w] = as_u64(acc);
                if (acc > 0.0) {
                    int ex;
                    frexp(acc, &ex);
                    my_maxe = max(my_maxe, ex);
                    my_mine = min(my_mine, ex);
                }
            }
        }
    } else if (phase == PH_BWD) {
        const int qb = s_qb, cnt = s_qe - s_qb;
        const int sh = s_sh0, shn = s_sh1;
        const bool dump = s_dump != 0;
        const int n_light = (cnt + kPer - 1) / kPer;
        const int total = n_light + hseg;
        for (int k = gw; k < total; k += nw) {
            const int it = k < hseg ? n_light + k : k - hseg;  // heavy segments first
            if (it >= n_light) {  // a segment of a heavy vertex of level l
                const int t = it - n_light;
                const int h = seg_owner(a.hq.seg, h0, h1, t);
                const int s = t - a.hq.seg[h];
                const int v = a.queue[a.hq.pos[h]];
                const int e0 = rp[v], e1 = rp[v + 1];
                const int a0 = seg_begin(a.g, e0, s), a1 = seg_end(a.g, e0, e1, s);
                const double p = plain_sum<kWave>(a, a0, a1 - a0, l + 1, true, 0, my_larcs);
                if (lane == 0) {
                    my_arcs += (unsigned)(a1 - a0);
                    part_store(&a.hq.part_lo[a.hq.seg[h] + s], as_u64(p));
                }
                const int ns = n_segments(a.g, e1 - e0);
                if (!seg_arrive(&a.hq.cnt[h], ns)) continue;
                if (lane == 0) {
                    double acc = 0.0;
                    for (int k = 0; k < ns; ++k) acc += as_f64(part_load(&a.hq.part_lo[a.hq.seg[h] + k]));
                    const double sv = norm_sigma<MODE>(a, v, sh);
                    double delta = sv * acc;
                    if (MODE == 1) delta = ldexp(delta, -shn);
                    a.chat[v] = (1.0 + delta) / sv;
                    a.bc[v] += delta;
                    if (dump) a.dump_delta[v] = delta;
                    a.hq.cnt[h] = 0;
                }
                continue;
            }
            const int i = it * kPer + sub;
            const bool valid = i < cnt;
            const int v = valid ? a.queue[qb + i] : 0;
            const int e0 = valid ? rp[v] : 0;
            const int deg = valid ? rp[v + 1] - e0 : 0;
            const bool fin = lead && valid && deg <= seg_arcs(a.g);
            const double sv = fin ? norm_sigma<MODE>(a, v, sh) : 1.0;
            const double bc0 = fin ? a.bc[v] : 0.0;
            if (lead) my_arcs += (unsigned)(deg <= seg_arcs(a.g) ? deg : 0);
            double acc = plain_sum<kSub>(a, e0, deg <= kSubDeg ? deg : 0, l + 1, true, 0, my_larcs);
            unsigned long long mm = __ballot(lead && deg > kSubDeg && deg <= seg_arcs(a.g));
            while (mm) {
                const int j = __ffsll(mm) - 1;
                mm &= mm - 1;
                const double p = plain_sum<kWave>(a, __shfl(e0, j), __shfl(deg, j), l + 1, true, 0, my_larcs);
                if (lane == j) acc = p;
            }
            if (fin) {
                double delta = sv * acc;
                if (MODE == 1) delta = ldexp(delta, -shn);
                a.chat[v] = (1.0 + delta) / sv;
                a.bc[v] = bc0 + delta;
                if (dump) a.dump_delta[v] = delta;
            }
        }
    } else if (phase == PH_FIN) {
        const int total = s_qe, next_src = s_sh0;
        for (int i = blockIdx.x * kBlock + tid; i < total; i += (int)nblk * kBlock) {
            const int v = a.queue[i];
            if (v == next_src) continue;
            d[v] = -1;
            sig[v] = 0ull;
        }
    } else if (phase == PH_DUMP_FWD) {
        for (int v = blockIdx.x * kBlock + tid; v < n; v += (int)nblk * kBlock) {
            a.dump_d[v] = d[v];
            a.dump_sig[v] = sig[v];
        }
        if (blockIdx.x == 0)
            for (int i = tid; i < c->n_levels; i += kBlock) a.dump_shift[i] = MODE ? a.shift[i] : 0;
    }

    // ---- per-launch counters into the slots; the last workgroup continues
    Counters cn;
    cn.v[SC_EDGES] = my_edges;
    cn.v[SC_ARCS] = my_arcs;
    cn.v[SC_LARCS] = my_larcs;
    cn.v[SC_OVF] = my_ovf ? 1ull : 0ull;
    if (my_maxe != INT_MIN) cn.exponent(my_maxe);
    if (my_mine != INT_MAX) cn.exponent(my_mine);
    if (!step_epilogue<kWavesPerBlock>(gc, cn, s_red, s_tot, &s_last, blockIdx.x, nblk)) return;

    // ---- the last workgroup advances the state machine
    int begin_pos = 0;
    int advance = 0;
    uint32_t cnt_next = 0;
    unsigned long long edges_next = 0;
    if (tid == 0) {
        c->st_steps += 1;
        c->st_arcs += s_tot[SC_ARCS];
        c->st_lane_arcs += s_tot[SC_LARCS];
        c->st_parcs[phase] += s_tot[SC_ARCS];
        c->st_plarcs[phase] += s_tot[SC_LARCS];
        c->st_ppairs[phase] += s_tot[SC_PAIRS];
        const unsigned long long now = wall_clock64();
        const unsigned long long dt = c->last_tick ? now - c->last_tick : 0ull;
        c->st_ticks[phase] += dt;
        if (phase == PH_FWD) c->st_vticks[s_variant] += dt;
        c->last_tick = now;
        const int rl = (phase == PH_FWD || phase == PH_BWD) ? l : (phase == PH_SIG ? l + 1 : -1);
        if (rl >= 0) {
            LevelRec &r = level_rec(a.lvl, rl);
            (void)atomicAdd(&r.arcs, s_tot[SC_ARCS]);
            (void)atomicAdd(&r.ticks, dt);
            if (phase == PH_FWD) {
                (void)atomicAdd(&r.visits, 1ull);
                (void)atomicAdd(&r.var[s_variant], 1ull);
            }
        }
        if (phase == PH_FWD) {
            const uint32_t cnt = (uint32_t)ld_agent(&gc->next_qc);
            const unsigned long long nh = ld_agent(&gc->next_hq);
            const int qe = s_qe;  // level_off[l + 1]
            a.level_off[l + 2] = qe + (int)cnt;
            a.hq.off[l + 2] = s_hqb + (int)(uint32_t)nh;
            a.hq.nseg[l + 1] = (int)(nh >> 32);
            gc->next_hq = 0;
            c->st_fwd_levels += 1;
            c->st_var[s_variant] += 1;
            c->st_qentries += cnt;
            c->st_lane_entries += cnt;
            (void)atomicAdd(&level_rec(a.lvl, l + 1).entries, (unsigned long long)cnt);
            if (MODE == 0 && s_tot[SC_OVF]) {
                const uint32_t k = c->n_ovf;
                if (k < a.ovf_cap) a.ovf_list[k] = c->pos;
                else gc->err |= ERR_OVF_CAP;
                c->n_ovf = k + 1;
                c->total_queued = (uint32_t)(qe + (int)cnt);
                c->phase = PH_FIN;
            } else if (cnt == 0) {
                c->total_queued = (uint32_t)qe;
                plain_after_forward(a, c, l + 1);
            } else if (MODE == 1) {
                c->phase = PH_SIG;
                c->next_edges = s_tot[SC_EDGES];  // kept for the level advance after the path counts
            } else {
                advance = 1;
                cnt_next = cnt;
                edges_next = s_tot[SC_EDGES];
            }
        } else if (phase == PH_SIG) {
            const bool any = s_tot[SC_MAXE] != 0;
            const int mx = (int)s_tot[SC_MAXE] - 4096, mn = 4096 - (int)s_tot[SC_MINE];
            int sh = 0;
            if (any && mx > kExpHigh) sh = mx - kExpTarget;
            if (any && mn - sh < kExpLow) gc->err |= ERR_SIGMA_RANGE;
            a.shift[l + 1] = sh;
            advance = 1;
            cnt_next = (uint32_t)ld_agent(&gc->next_qc);
            edges_next = c->next_edges;
        } else if (phase == PH_BWD) {
            if (l - 1 >= 1) {
                c->level = l - 1;
            } else {
                c->total_queued = (uint32_t)a.level_off[c->n_levels];
                c->phase = PH_FIN;
            }
        } else if (phase == PH_DUMP_FWD) {
            c->dump_state = 1;
            const int L = c->n_levels;
            if (L >= 2) {
                c->phase = PH_BWD;
                c->level = L - 1;
            } else {
                c->phase = PH_FIN;
            }
        } else if (phase == PH_FIN) {
            if (c->dump_state == 1 && c->dump_pos == c->pos) c->dump_state = 2;
            const int64_t next = c->pos + 1;
            c->pos = next;
            if (next < c->n_items) begin_pos = 1;
            else c->phase = PH_DONE;
        }
        s_qb = begin_pos;
        s_qe = advance;
        s_qn = (int)cnt_next;
        s_red[0] = edges_next;
    }
    __syncthreads();
    if (s_qb == 1) plain_begin_source<MODE>(a, gc, c, c->pos, s_lds, &s_feat);
    else if (s_qe == 1) plain_advance_level<MODE>(a, gc, c, l, (uint32_t)s_qn, s_red[0], s_lds, &s_feat);
    head_store(gc, s_head, a.parity);
}

template __global__ void plain_step<0>(PlainArgs);
template __global__ void plain_step<1>(PlainArgs);

}  // namespace bcx
