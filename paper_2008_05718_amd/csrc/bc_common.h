// bc_common.h -- wavefront helpers and the per-level policy, shared by the
// plain and batched step kernels.  Internal to libbc.
#pragma once

#include <climits>
#include <cmath>

#include "bc_dev.h"

namespace bcx {

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Number of set bits of m below this lane.
__device__ __forceinline__ unsigned lanes_below(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// A value that is the same in every lane, moved to a scalar register: loop
// bounds and branches on it then need no change of the execution mask.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ unsigned long long uniform(unsigned long long x) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)x);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(x >> 32));
    return ((unsigned long long)hi << 32) | lo;
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}
__device__ __forceinline__ unsigned long long wave_or_u64(unsigned long long x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x |= __shfl_xor(x, o);
    return x;
}
// Butterfly sum: a fixed association, so every lane ends with the same bits
// and the result does not depend on anything but the 64 inputs.
__device__ __forceinline__ double wave_sum_f64(double x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

__device__ __forceinline__ double as_f64(unsigned long long u) { return __longlong_as_double((long long)u); }
__device__ __forceinline__ unsigned long long as_u64(double x) { return (unsigned long long)__double_as_longlong(x); }

// ---------------------------------------------------------------- counters
struct Counters {
    unsigned long long v[kNCnt];
    __device__ Counters() {
#pragma unroll
        for (int k = 0; k < kNCnt; ++k) v[k] = 0ull;
    }
    __device__ void exponent(int e) {
        v[SC_MAXE] = max(v[SC_MAXE], (unsigned long long)(e + 4096));
        v[SC_MINE] = max(v[SC_MINE], (unsigned long long)(4096 - e));
    }
};

__device__ __forceinline__ int cnt_op(int k) {  // 0 sum, 1 or, 2 max
    return k >= SC_PAIRS ? 0 : (k >= SC_MAXE ? 2 : (k >= SC_ACT ? 1 : 0));
}

__device__ __forceinline__ unsigned long long cnt_combine(int k, unsigned long long a, unsigned long long b) {
    const int op = cnt_op(k);
    return op == 0 ? a + b : (op == 1 ? (a | b) : (a > b ? a : b));
}

// Workgroups a step needs for `items` wavefront work items (at least one, at
// most the launched grid).  Workgroups beyond it leave at once.
__device__ __forceinline__ unsigned active_blocks(long long items, unsigned grid) {
    long long b = (items + kWavesPerBlock - 1) / kWavesPerBlock;
    if (b < 1) b = 1;
    if (b > (long long)grid) b = grid;
    return (unsigned)b;
}

// Work items of a step, [0, total), are dealt to ncls = min(nblk, kSlots)
// classes k mod ncls; the workgroups of class r (blockIdx.x mod ncls) share
// that class's items: each wavefront takes its first one statically, later
// ones from the class's counter (reset by the last workgroup of the launch),
// so a wavefront that finishes early takes the next item without all
// wavefronts meeting on one address.  Items are independent and each sum
// stays inside one item, so the assignment never changes a result.
template <int NW = kWavesPerBlock>
struct WorkCursor {
    uint32_t *ctr;
    int r, ncls, nwr, j, jn;
    template <class C>
    __device__ __forceinline__ WorkCursor(C *c, unsigned nblk, unsigned bid) {
        ncls = (int)(nblk < (unsigned)kSlots ? nblk : (unsigned)kSlots);
        r = (int)(bid % (unsigned)ncls);
        const int nb = ((int)nblk - r + ncls - 1) / ncls;  // workgroups of class r
        nwr = nb * NW;
        j = (int)(bid / (unsigned)ncls) * NW + uniform((int)(threadIdx.x >> 6));
        ctr = &c->work[r][0];
        jn = fetch();
    }
    __device__ __forceinline__ int fetch() {
        int x = 0;
        if ((threadIdx.x & 63) == 0) x = (int)atomicAdd(ctr, 1u);
        return nwr + uniform(x);
    }
    __device__ __forceinline__ int item() const { return r + ncls * j; }
    __device__ __forceinline__ void next(int total) {
        j = jn;
        if (item() < total) jn = fetch();
    }
};

// Copy of the state in LDS: one 8-byte load per thread and one round trip
// (field by field, every update by the last workgroup's one thread stood behind
// a load of its own: about 10 us of a step).
template <int NT>
__device__ __forceinline__ void head_load(Head &s, const Head &g) {
    unsigned long long *d = (unsigned long long *)&s;
    const unsigned long long *p = (const unsigned long long *)&g;
    for (int i = threadIdx.x; i < (int)(sizeof(Head) / 8); i += NT) d[i] = p[i];
}
// The next state, for the launch of the other parity (last workgroup, all
// threads).  Workgroups without work may still be reading the current one.
__device__ __forceinline__ void head_store(Ctl *c, const Head &s, int parity) {
    __syncthreads();
    const unsigned long long *p = (const unsigned long long *)&s;
    unsigned long long *d = (unsigned long long *)&c->h[1 - parity];
    for (int i = threadIdx.x; i < (int)(sizeof(Head) / 8); i += kBlock) d[i] = p[i];
    if (threadIdx.x == 0) {
        c->phase = s.phase;
        if (s.phase == PH_DONE) c->h[parity].phase = PH_DONE;
    }
}

// End of a step for one workgroup that took part: reduce the counters over
// the workgroup, add them into the workgroup's slot, count the workgroup in
// (two-level arrival so no single address takes one atomic per workgroup).
// Returns true in exactly one workgroup -- the last -- once the nblk workgroups
// that take part have arrived; s_tot then holds the totals, and slots, arrival
// and work counters are reset.
//
// No fences: within a launch, workgroups exchange only device-scope atomics
// here (slot counters, arrival counts, queue counters); plain stores are
// consumed by later launches, which kernel boundaries order.  The last
// workgroup must therefore never store to a word that another workgroup of
// the same launch stored to: each XCD's L2 would hold its own dirty copy
// until the launch ends and write it back in no fixed order.  Device-scope
// atomics that a workgroup issues before calling this (the slot counters
// here, a caller's exponent ranges) must have completed before it counts
// itself in: each wave that issued one waits for its memory counters first.
// A step of one workgroup (nblk = 1) exchanges nothing.
// s_red needs NW * kNCnt entries.  mlp: weights the last workgroup will need, or
// nullptr.
template <int NW, class C>
__device__ __forceinline__ bool step_epilogue(C *c, Counters &cn, unsigned long long *s_red, unsigned long long *s_tot,
                                              int *s_last, unsigned bid, unsigned nblk, const float *mlp = nullptr) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < kNCnt; ++k) {
        unsigned long long x = cn.v[k];
        if (__any(x != 0ull)) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) x = cnt_combine(k, x, __shfl_xor(x, o));
        }
        if (lane == 0) s_red[wid * kNCnt + k] = x;
    }
    __syncthreads();
    unsigned long long t = 0;
    const int k = threadIdx.x;
    if (k < kNCnt) {
        t = s_red[k];
        for (int w = 1; w < NW; ++w) t = cnt_combine(k, t, s_red[w * kNCnt + k]);
    }
    if (nblk == 1) {
        if (k < kNCnt) s_tot[k] = t;
        if (k == 0) c->work[0][0] = 0u;
        __syncthreads();
        return true;
    }
    if constexpr (NW == kWavesPerBlock && sizeof(C) == sizeof(Ctl)) {
        const int slot = bid % kSlots;
        if (k < kNCnt && t) {
            const int op = cnt_op(k);
            if (op == 0) atomicAdd(&c->slot[slot][k], t);
            else if (op == 1) atomicOr(&c->slot[slot][k], t);
            else atomicMax(&c->slot[slot][k], t);
        }
        // The slot atomics return nothing, so nothing has waited for them;
        // the last workgroup reads the slots once every arrival is counted,
        // so they must have completed before this workgroup arrives.
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __syncthreads();
        const unsigned nslots = nblk < (unsigned)kSlots ? nblk : (unsigned)kSlots;
        if (threadIdx.x == 0) {
            int last = 0;
            const unsigned in_slot = (nblk - slot + kSlots - 1) / kSlots;
            if (atomicAdd(&c->arrive[slot][0], 1u) == in_slot - 1)
                last = atomicAdd(&c->blocks_done, 1u) == nslots - 1 ? 1 : 0;
            *s_last = last;
        }
        __syncthreads();
        if (!*s_last) return false;
        // the policy network's weights into this XCD's L2 while the totals are on
        // their way (a word of every 64 bytes)
        float near = 0.0f;
        if (mlp && (int)threadIdx.x * 16 < kMlpParams) near = mlp[threadIdx.x * 16];
        // totals: wavefront w takes counters w, w + 4, ..., lane = slot
        unsigned long long x[(kNCnt + NW - 1) / NW];
#pragma unroll
        for (int q = 0; q < (kNCnt + NW - 1) / NW; ++q) {
            const int kk = wid + q * NW;
            x[q] = (kk < kNCnt && lane < (int)nslots)
                       ? __hip_atomic_load(&c->slot[lane][kk], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                       : 0ull;
        }
#pragma unroll
        for (int q = 0; q < (kNCnt + NW - 1) / NW; ++q) {
            const int kk = wid + q * NW;
            if (kk >= kNCnt) break;
            unsigned long long y = x[q];
#pragma unroll
            for (int o = kSlots / 2; o > 0; o >>= 1) y = cnt_combine(kk, y, __shfl_xor(y, o));
            if (lane == 0) s_tot[kk] = y;
            if (lane < (int)nslots) c->slot[lane][kk] = 0ull;
        }
        if (threadIdx.x < nslots) {
            c->arrive[threadIdx.x][0] = 0u;
            c->work[threadIdx.x][0] = 0u;
        }
        if (threadIdx.x == 0) c->blocks_done = 0u;
        asm volatile("" ::"v"(near));
        __syncthreads();
    }
    return true;
}

// ----------------------------------------------------------- staged appends
// New level-queue entries are first gathered per wavefront in LDS and
// written in runs, one position atomic per run instead of per append.
// A vertex's degree is looked up when its run is written (vertex by vertex, that
// lookup stood behind every atomic that found one) and kept as cost units, 0
// for a heavy one.
constexpr int kStage = 288;
struct Stage {
    int32_t w[kStage];
    uint8_t cost[kStage];
};
// What a workgroup's last runs take together.
template <int NW>
struct StageTotals {
    unsigned n[NW], cost[NW];
    unsigned long long at;
};

// Wavefront-inclusive prefix sum of an int, by the data-parallel row shifts and
// broadcasts (no LDS traffic): within rows of 16, then row 0 into 1 and 2
// into 3, then the lower half into the upper.  All lanes take part.
__device__ __forceinline__ int wave_incl_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
    return x;
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ unsigned wave_sum_u32(unsigned x) {
    return (unsigned)__builtin_amdgcn_readlane(wave_incl_scan((int)x), 63);
}

__device__ __forceinline__ unsigned long long shfl_u64(unsigned long long x, int src) {
    const unsigned lo = __shfl((unsigned)x, src), hi = __shfl((unsigned)(x >> 32), src);
    return ((unsigned long long)hi << 32) | lo;
}

__device__ __forceinline__ int seg_arcs(const GraphArgs &g) { return 1 << g.seg_log; }
__device__ __forceinline__ int n_segments(const GraphArgs &g, int deg) {
    return (int)(((unsigned)deg + (unsigned)seg_arcs(g) - 1u) >> g.seg_log);
}

// Segment s of a row [e0, e1): its first arc and its end (the same where the row
// has fewer segments).  A row may end at 2^31 - 1, so nothing is added to a
// position before it is known that the row goes on: sums over a row's
// arcs count from its first one, and a segment's arcs are what is left of the row.
__host__ __device__ __forceinline__ constexpr int seg_len(int left, int s, int seg_log) {
    const int l = left - (int)((unsigned)s << seg_log);
    return l < 0 ? 0 : l < (1 << seg_log) ? l : 1 << seg_log;
}
static_assert(seg_len(1024, 0, 10) == 1024 && seg_len(1025, 0, 10) == 1024 && seg_len(1025, 1, 10) == 1 &&
                  seg_len(5, 1, 10) == 0 && seg_len(INT_MAX, 0, 10) == 1024 && seg_len(INT_MAX, (INT_MAX >> 10), 10) == 1023,
              "a row's last segment is what is left of it");
__device__ __forceinline__ int seg_begin(const GraphArgs &g, int e0, int s) {
    return (int)((unsigned)e0 + ((unsigned)s << g.seg_log));
}
__device__ __forceinline__ int seg_end(const GraphArgs &g, int e0, int e1, int s) {
    return seg_begin(g, e0, s) + seg_len(e1 - e0, s, g.seg_log);
}

// Degree that decides how a level entry is processed (one thread, one
// wavefront, or segments) and what it costs: the larger of its out-
// and in-degree, so an entry is handled the same way in every phase, whichever
// arcs the phase scans (out-arcs to push and to pull dependencies from
// successors, in-arcs to pull discovery and path counts from predecessors).
// For an undirected graph it is the degree.
__device__ __forceinline__ int class_deg(const GraphArgs &g, int v, int out_deg) {
    return g.directed ? max(out_deg, g.in_row_ptr[v + 1] - g.in_row_ptr[v]) : out_deg;
}


#ifndef BC_BUDGET
#define BC_BUDGET 16
#endif
constexpr int kBudget = BC_BUDGET;  // cost units (8 arcs each) per work group
#ifndef BC_MERGE
#define BC_MERGE 8
#endif
constexpr int kMergeMax = BC_MERGE;  // consecutive groups a wavefront takes at once on large levels
static_assert(kBudget >= 2 && kBudget * kMergeMax <= 128, "a merged group must fit in one wavefront (every entry costs >= 2 units)");
// Groups per item of a step with ng groups on `waves` wavefronts: each wavefront
// gets one item while the level is small, items of full size beyond (a group
// costs a wavefront its entries' offsets and words before the first arc).
__device__ __forceinline__ int merge_groups(uint32_t ng, unsigned waves) {
    return (int)min((uint32_t)kMergeMax, max(1u, (ng + waves - 1) / waves));
}

// Work estimate of a level entry in units of 8 arcs: its adjacency plus a
// fixed part; heavy entries (split into segments elsewhere) count 2.  Every
// entry costs at least 2 units, so a group never holds more than
// kBudget / 2 entries.
static __host__ __device__ __forceinline__ unsigned entry_cost(int deg, int seg_log) {
    return deg > (1 << seg_log) ? 2u : 1u + (unsigned)(deg + 7) / 8u;
}

// Groups of a level: the entries whose cost prefix (in append order) starts
// in [k * kBudget, (k + 1) * kBudget) form group k, so every group carries
// about the same work.  Groups are found through gstart: gstart[gb + k] is
// the level-relative index of group k's first entry.  An entry whose cost
// range (P, P + c] contains the boundary k * kBudget writes gstart[gb + k] =
// its index + 1; gstart[gb] = 0 and the end are set when the level closes.
struct GroupArgs {
    uint32_t *gstart = nullptr;  // nullptr: no groups (per-source engine)
    uint32_t gb = 0;             // first gstart slot of the level being appended
    uint32_t gcap = 0;
};

// Where an engine's next level is appended; deg(w, first) is the degree that
// classifies vertex w (first: asked for the first time).
template <class C, class Deg>
struct StageTo {
    C *c;
    int32_t *q;
    uint32_t qbase, qcap;
    HeavyQ hq;
    uint32_t hq_base;
    GroupArgs ga;
    const GraphArgs &g;
    Deg deg;
};
template <class C, class Deg>
__device__ __forceinline__ StageTo<C, Deg> stage_to(C *c, int32_t *q, uint32_t qbase, uint32_t qcap, const HeavyQ &hq,
                                                    uint32_t hq_base, const GroupArgs &ga, const GraphArgs &g,
                                                    Deg deg) {
    return StageTo<C, Deg>{c, q, qbase, qcap, hq, hq_base, ga, g, deg};
}

__device__ __forceinline__ void stage_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Degrees of the n staged entries; returns their cost units.
template <class To>
__device__ __forceinline__ unsigned stage_costs(Stage &st, int n, const To &to) {
    stage_fence();
    unsigned cost = 0;
    for (int i = lane_id(); i < n; i += kWave) {
        const int deg = to.deg(st.w[i], true);
        const unsigned ci = entry_cost(deg, to.g.seg_log);
        st.cost[i] = deg > seg_arcs(to.g) ? (uint8_t)0 : (uint8_t)ci;
        cost += ci;
    }
    static_assert(1 + (kSegMax + 7) / 8 <= 255, "cost units of an entry fit a byte");
    return wave_sum_u32(cost);
}

// Write the n staged entries of this wavefront to the level queue (positions
// qbase + base and on, cost units from cbase on), heavy ones also to the
// level's heavy list.
template <class To>
__device__ __forceinline__ void stage_write(Stage &st, int n, unsigned base, unsigned cbase, const To &to) {
    stage_fence();
    const int lane = lane_id();
    for (int i0 = 0; i0 < n; i0 += kWave) {
        const int i = i0 + lane;
        const bool on = i < n;
        const int w = on ? st.w[i] : 0;
        const unsigned units = on ? st.cost[i] : 1u;
        const bool heavy = on && units == 0u;
        const uint32_t p = to.qbase + base + (uint32_t)i;
        if (on) {
            if (p < to.qcap) to.q[p] = w;
            else atomicOr(&to.c->err, ERR_QUEUE_CAP);
        }
        if (to.ga.gstart) {
            const unsigned ci = heavy ? 2u : on ? units : 0u;
            const unsigned incl = (unsigned)wave_incl_scan((int)ci);
            const unsigned P = cbase + incl - ci;
            for (unsigned k = P / kBudget + 1; on && k <= (P + ci) / kBudget; ++k) {
                const unsigned long long at = (unsigned long long)to.ga.gb + k;
                if (at < to.ga.gcap) to.ga.gstart[at] = base + (uint32_t)i + 1u;
                else atomicOr(&to.c->err, ERR_QUEUE_CAP);
            }
            cbase += (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
        }
        const unsigned long long hm = __ballot(heavy);
        if (hm) {
            const int ns = heavy ? n_segments(to.g, to.deg(w, false)) : 0;
            const int incl = wave_incl_scan(ns);
            const int total = __builtin_amdgcn_readlane(incl, 63);
            const int hl = __ffsll((unsigned long long)hm) - 1;
            unsigned long long hold = 0;
            if (lane == hl)
                hold = atomicAdd(&to.c->next_hq,
                                 (unsigned long long)__popcll(hm) | ((unsigned long long)(unsigned)total << 32));
            hold = shfl_u64(hold, hl);
            if (heavy) {
                const uint32_t idx = to.hq_base + (uint32_t)hold + lanes_below(hm);
                if (idx < to.hq.cap) {
                    to.hq.pos[idx] = (int32_t)p;
                    to.hq.seg[idx] = (int32_t)(hold >> 32) + (incl - ns);
                    to.hq.cnt[idx] = 0;
                } else {
                    atomicOr(&to.c->err, ERR_QUEUE_CAP);
                }
            }
        }
    }
}

// A run's entries and cost units are taken by one 64-bit atomic.
template <class To>
__device__ __forceinline__ unsigned long long stage_take(unsigned n, unsigned cost, const To &to) {
    return atomicAdd(&to.c->next_qc, (unsigned long long)n | ((unsigned long long)(to.ga.gstart ? cost : 0u) << 32));
}

// Stage w for every lane with pred; a run is written once there is no room for
// another 64.  n is the wavefront-uniform fill count.  The wavefront must be
// converged.
template <class To>
__device__ __forceinline__ void stage_push(bool pred, int32_t w, Stage &st, int &n, const To &to) {
    const unsigned long long m = __ballot(pred);
    if (m == 0) return;
    if (pred) st.w[n + (int)lanes_below(m)] = w;
    n += __popcll(m);
    if (n <= kStage - kWave) return;
    const unsigned cost = stage_costs(st, n, to);
    unsigned long long at = 0;
    if (lane_id() == 0) at = stage_take((unsigned)n, cost, to);
    at = shfl_u64(at, 0);
    stage_write(st, n, (unsigned)at, (unsigned)(at >> 32), to);
    n = 0;
}

// Write what the workgroup's wavefronts have staged at the end of a step, with
// one atomic for all of them (all threads of the workgroup).  One per
// wavefront, on the same word, bounded every step that ran on many: 66 us for
// a pull level on R-MAT 18 with one source, now 50.
template <int NW, class To>
__device__ __forceinline__ void stage_finish(Stage &st, int n, StageTotals<NW> &tot, const To &to) {
    const int wid = uniform((int)(threadIdx.x >> 6));
    const unsigned cost = n ? stage_costs(st, n, to) : 0u;
    if (lane_id() == 0) {
        tot.n[wid] = (unsigned)n;
        tot.cost[wid] = cost;
    }
    __syncthreads();
    unsigned base = 0, cbase = 0, all = 0, call = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        if (w == wid) {
            base = all;
            cbase = call;
        }
        all += tot.n[w];
        call += tot.cost[w];
    }
    if (threadIdx.x == 0 && all) tot.at = stage_take(all, call, to);
    __syncthreads();
    if (n) stage_write(st, n, (unsigned)tot.at + base, (unsigned)(tot.at >> 32) + cbase, to);
}

// Largest h in [h0, h1) with seg[h] <= t (seg ascending, seg[h0] = 0 <= t).
__device__ __forceinline__ int seg_owner(const int32_t *seg, int h0, int h1, int t) {
    int lo = h0, hi = h1;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (seg[mid] <= t) lo = mid;
        else hi = mid;
    }
    return lo;
}

// First index i in [0, n) with a[i] >= x (a ascending).
__device__ __forceinline__ int lower_bound_i32(const int32_t *a, int n, int x) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Features of a level, normalised as documented for the policy network.
struct LevelFeatures {
    float nf, mf, nu, mu;
    int level;
};

__device__ __forceinline__ void mlp_inputs(const LevelFeatures &f, float n, float nnz, float *x) {
    const float ln = log2f(1.0f + n), lm = log2f(1.0f + nnz);
    x[0] = log2f(1.0f + f.nf) / fmaxf(ln, 1.0f);
    x[1] = log2f(1.0f + f.mf) / fmaxf(lm, 1.0f);
    x[2] = log2f(1.0f + f.nu) / fmaxf(ln, 1.0f);
    x[3] = log2f(1.0f + f.mu) / fmaxf(lm, 1.0f);
    x[4] = (float)f.level / 64.0f;
}

// Direction-optimising rule (Beamer, Asanovic, Patterson, SC'12): go
// bottom-up once the frontier's arcs exceed the unvisited arcs / alpha, come
// back top-down once the frontier has fewer than n / beta vertices.  The
// push variants split by mean frontier degree.
__device__ __forceinline__ int heuristic_variant(const PolicyArgs &p, int prev, const LevelFeatures &f,
                                                 float n) {
    bool pull;
    if (prev == V_PULL) pull = !(f.nf < n / p.beta);
    else pull = f.mf > f.mu / p.alpha;
    if (pull) return V_PULL;
    return (f.nf > 0.0f && f.mf / f.nf > p.wpv_degree) ? V_PUSH_WPV : V_PUSH_TPV;
}

// argmin of y[k0 .. k0 + 2] (the first on ties)
__device__ __forceinline__ int argmin3(const float *y, int k0) {
    int best = 0;
    float bv = y[k0];
    if (y[k0 + 1] < bv) { best = 1; bv = y[k0 + 1]; }
    if (y[k0 + 2] < bv) best = 2;
    return best;
}

// Choose the variant of the next level, and (in *lbo) the summation options
// of the path-count step that sums the entries it discovers and of the
// backward step over the level's own entries (option | option << 2).  Called
// by every thread of one workgroup (the MLP spreads its hidden units over
// threads); the result is returned to every thread.  lds needs
// 2 * kMlpH + kMlpOut floats.  Only the learned policy changes the summation
// options; every other policy keeps the sources-per-entry rule.
__device__ __forceinline__ int choose_variant(const PolicyArgs &p, int policy, int prev, const LevelFeatures &f, float n,
                              float nnz, float *lds, int *lbo) {
    *lbo = kLbDefault;
    if (policy == POL_FORCE_TPV) return V_PUSH_TPV;
    if (policy == POL_FORCE_WPV) return V_PUSH_WPV;
    if (policy == POL_FORCE_PULL) return V_PULL;
    if (policy == POL_MLP && p.has_mlp) {
        const float *W1 = p.mlp;
        const float *b1 = W1 + kMlpH * kMlpIn;
        const float *W2 = b1 + kMlpH;
        const float *b2 = W2 + kMlpH * kMlpH;
        const float *W3 = b2 + kMlpH;
        const float *b3 = W3 + kMlpOut * kMlpH;
        // Eight threads to a unit of the later layers, and every weight requested
        // before the first layer: layer by layer, row by row in one thread,
        // this stood with three rounds of 32 loads at the end of every forward
        // step (with the choices of the rule, R-MAT 2^16, 512 sources: 2.1 % of the run, now 1.0).
        static_assert(kMlpH == 32 && kMlpOut <= 32, "eight threads hold a row of weights, four each");
        const int t = threadIdx.x, u = t >> 3, q = t & 7;
        float w1[kMlpIn], c1 = 0.0f, c2 = 0.0f, c3 = 0.0f;
        float4 w2 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), w3 = w2;
        if (t < kMlpH) {
            for (int i = 0; i < kMlpIn; ++i) w1[i] = W1[t * kMlpIn + i];
            c1 = b1[t];
        }
        if (u < kMlpH) {
            w2 = *reinterpret_cast<const float4 *>(W2 + u * kMlpH + 4 * q);
            c2 = b2[u];
        }
        if (u < kMlpOut) {
            w3 = *reinterpret_cast<const float4 *>(W3 + u * kMlpH + 4 * q);
            c3 = b3[u];
        }
        float x[kMlpIn];
        mlp_inputs(f, n, nnz, x);
        float *h1 = lds, *h2 = lds + kMlpH, *y = lds + 2 * kMlpH;
        auto row = [&](const float4 &w, const float *h) {
            float s = w.x * h[4 * q] + w.y * h[4 * q + 1] + w.z * h[4 * q + 2] + w.w * h[4 * q + 3];
            // sums over eight threads: neighbours, pairs, then the half row mirrored
            s += dpp_f32<0xB1>(s);
            s += dpp_f32<0x4E>(s);
            return s + dpp_f32<0x141>(s);
        };
        if (t < kMlpH) {
            float s = c1;
            for (int i = 0; i < kMlpIn; ++i) s += w1[i] * x[i];
            h1[t] = fmaxf(s, 0.0f);
        }
        __syncthreads();
        const float s2 = row(w2, h1) + c2;
        if (u < kMlpH && q == 0) h2[u] = fmaxf(s2, 0.0f);
        __syncthreads();
        const float s3 = row(w3, h2) + c3;
        if (u < kMlpOut && q == 0) y[u] = s3;
        __syncthreads();
        float yy[kMlpOut];
        bool finite = true;
        for (int k = 0; k < kMlpOut; ++k) {
            yy[k] = y[k];
            finite = finite && isfinite(yy[k]);
        }
        __syncthreads();
        if (finite) {
            // the rule's choice stands unless the network predicts a gain of
            // at least p.margin (log2 units) for another one
            const float m = p.margin;
            int v = argmin3(yy, kOutFwd), so = argmin3(yy, kOutSig), bo = argmin3(yy, kOutBwd);
            const int h = heuristic_variant(p, prev, f, n);
            if (yy[kOutFwd + h] - yy[kOutFwd + v] < m) v = h;
            if (yy[kOutSig + LB_RULE] - yy[kOutSig + so] < m) so = LB_RULE;
            if (yy[kOutBwd + LB_RULE] - yy[kOutBwd + bo] < m) bo = LB_RULE;
            *lbo = so | (bo << 2);
            return v;
        }
        // non-finite prediction: fall back to the rules
    }
    return heuristic_variant(p, prev, f, n);
}

// Sources-per-entry threshold of a summation option: groups whose light
// entries carry at most this many sources on average are summed by (entry,
// source) pairs.
__device__ __forceinline__ float lb_item_lanes(const PolicyArgs &p, int opt) {
    return opt == LB_PACKED ? -1.0f : (opt == LB_ITEMS ? 65.0f : p.item_lanes);
}

// Partial sums exchanged between the wavefronts of one launch (segments of
// a heavy vertex): stored and loaded with device-scope relaxed atomics, which
// are written through to, and read from, the point of coherence of all
// XCDs, so no cache-wide fence (L2 write-back / invalidate) is needed.
// seg_arrive waits until this wavefront's partial stores have completed,
// then counts it in; the wavefront that arrives last (returns true) reads
// every partial with part_load.
__device__ __forceinline__ void part_store(unsigned long long *p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long part_load(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool seg_arrive(int32_t *cnt, int nseg) {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);  // every memory operation of this wavefront has completed
    int old = 0;
    if (lane_id() == 0) old = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    old = __shfl(old, 0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    return old == nseg - 1;
}

template <typename T>
__device__ __forceinline__ T ld_agent(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace bcx
