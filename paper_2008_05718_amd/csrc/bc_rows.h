// bc_rows.h -- sums over adjacency lists in which every matched far end
// contributes a row of per-source values: the path counts and dependencies
// of the batched engines.  The including file defines bcx::kUnroll, the
// matches whose rows are loaded together.  Internal to libbc.
#pragma once

#include "bc_common.h"

namespace bcx {

// Per-source values live in vertex-major slabs [n][64]: path count, c and
// delta of vertex v for lane k at v * 64 + k.  Each (vertex, lane) pair is on
// exactly one level of a batch, so the slot is written once per batch and
// read only through a matching level tag and lane mask; nothing is cleared.
__device__ __forceinline__ unsigned long long readlane_u64(unsigned long long x, int j) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, j);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(x >> 32), j);
    return ((unsigned long long)hi << 32) | lo;
}

// A slab row read or written for the lanes of a wavefront-uniform mask: the
// row is a buffer of 512 bytes whose address sits in scalar registers, and a
// lane outside the mask takes an offset outside the buffer, for which loads
// return zero and stores do nothing (the buffer instructions' range check).
// A masked row access is then one select and one memory instruction: no
// change of the execution mask, no branch, no zeroed register.
constexpr unsigned kNoSlot = 0xfffffff0u;
constexpr int kRowBytes = kLanes * 8;
typedef unsigned row_data __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned row_slot(unsigned long long m) {
    return __builtin_amdgcn_inverse_ballot_w64(m) ? (unsigned)lane_id() * 8u : kNoSlot;
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_at(unsigned long long addr) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)addr, 0, kRowBytes, 0x00020000);
}
__device__ __forceinline__ unsigned long long row_load(unsigned long long addr, unsigned slot) {
    const row_data d = __builtin_amdgcn_raw_buffer_load_b64(row_at(addr), (int)slot, 0, 0);
    return ((unsigned long long)d.y << 32) | d.x;
}
__device__ __forceinline__ void row_store(unsigned long long addr, unsigned slot, unsigned long long v) {
    row_data d;
    d.x = (unsigned)v;
    d.y = (unsigned)(v >> 32);
    __builtin_amdgcn_raw_buffer_store_b64(d, row_at(addr), (int)slot, 0, 0);
}
__device__ __forceinline__ unsigned long long row_addr(const void *slab, int v, int shift = 9) {
    return (unsigned long long)slab + ((unsigned long long)(unsigned)v << shift);
}
// A slab and the binary logarithm of its rows' bytes (a row may hold fewer
// than 64 sources; lanes beyond it are in no mask).
struct Slab {
    const void *p;
    int shift;
    __device__ __forceinline__ Slab(const void *p_, int shift_ = 9) : p(p_), shift(shift_) {}
    __device__ __forceinline__ unsigned long long row(int v) const { return row_addr(p, v, shift); }
};

// A frontier word in one 16-byte load (tag and mask together).
__device__ __forceinline__ unsigned long long tagged_lanes(const Tagged *fw, int u, uint32_t T, unsigned long long m) {
    const uint4 f = *reinterpret_cast<const uint4 *>(fw + u);
    return f.z == T ? ((((unsigned long long)f.y << 32) | f.x) & m) : 0ull;
}
// Which lanes of m an arc e to far end u contributes to: the far end's lanes
// on the level with tag T ...
struct TagLanes {
    const Tagged *fw;
    uint32_t T;
    __device__ __forceinline__ unsigned long long operator()(int, int u, unsigned long long m) const {
        return tagged_lanes(fw, u, T, m);
    }
};
// ... or the lanes recorded for the arc itself (shortest-path arcs of a
// weighted graph).
struct ArcLanes {
    const unsigned long long *arc;
    __device__ __forceinline__ unsigned long long operator()(int e, int, unsigned long long m) const {
        return arc[e] & m;
    }
};

// What a path-count or backward sum adds up, in the order of the arcs.
enum : int { OP_U64 = 0, OP_F64 = 1, OP_C = 2 };
template <int OP>
struct RowSum {
    unsigned long long lo = 0;  // OP_U64: 64-bit sum and its carries (fewer than 2^31 terms)
    unsigned hi = 0;
    double d = 0.0;             // OP_F64: counts scaled by 2^-sh; OP_C: c values
    __device__ __forceinline__ void add(unsigned long long v, int sh) {
        if (OP == OP_U64) {
            lo += v;
            hi += (lo < v) ? 1u : 0u;
        } else if (OP == OP_F64) {
            d += ldexp(as_f64(v), -sh);
        } else {
            d += as_f64(v);
        }
    }
    __device__ __forceinline__ void clear() {
        lo = 0;
        hi = 0;
        d = 0.0;
    }
};

// The rows of up to kUnroll matches of a chunk (bal: lanes whose arc's far
// end matches, in arc order; xj: its lanes; rj: its row; ownj: the group entry
// of the arc) are requested together, then handed to use(value, owner) in arc
// order.  Everything but the values is wavefront-uniform; a slot beyond the
// last match loads nothing (its value is zero) and repeats the owner before.
template <class Use>
__device__ __forceinline__ void take_matches(unsigned long long &bal, unsigned long long xj, unsigned long long rj,
                                             int ownj, Use use) {
    unsigned long long val[kUnroll];
    int own[kUnroll];
    static_assert(kUnroll % 4 == 0, "matches are taken four at a time");
#pragma unroll
    for (int h = 0; h < kUnroll; h += 4) {
        own[h] = -1;
        if (h && !bal) continue;
#pragma unroll
        for (int q = h; q < h + 4; ++q) {
            const int j = bal ? __ffsll(bal) - 1 : 0;
            const unsigned long long x = bal ? readlane_u64(xj, j) : 0ull;
            own[q] = bal ? __builtin_amdgcn_readlane(ownj, j) : own[q > h ? q - 1 : h];
            bal &= bal - 1;
            val[q] = row_load(readlane_u64(rj, j), row_slot(x));
        }
    }
#pragma unroll
    for (int h = 0; h < kUnroll; h += 4) {
        if (h && own[h] < 0) break;
#pragma unroll
        for (int q = h; q < h + 4; ++q) use(val[q], own[q]);
    }
}

// Counters of a wavefront's path-count or backward items.
struct ArcCounters {
    unsigned larcs = 0, arcs = 0, pairs = 0;
};

// Sum over arcs [a0, a1) (one entry's, wavefront-uniform bounds) of the rows
// of the far ends, for the lanes of m that `lanes` gives each arc; lane k
// accumulates source k's value in CSR order.  The next chunk's frontier words and the
// column indices after them are requested before this chunk's rows.
template <int OP, class Lanes>
__device__ __forceinline__ void row_arcs(Lanes lanes, unsigned long long m, int a0, int a1, int sh,
                                         const int32_t *__restrict__ col, Slab slab, RowSum<OP> &acc,
                                         ArcCounters &ac) {
    if (a0 >= a1) return;
    const int lane = lane_id(), n = a1 - a0;
    col += a0;
    int u = col[min(lane, n - 1)];
    int un = col[min(kWave + lane, n - 1)];
    unsigned long long f = lanes(a0 + min(lane, n - 1), u, m);
    unsigned larcs = 0, pairs = 0;
    for (int i = 0; i < n; i += kWave) {
        const unsigned long long xj = i + lane < n ? f : 0ull;
        const unsigned long long rj = slab.row(u);
        unsigned long long bal = __ballot(xj != 0ull);
        if (i + kWave < n) {
            u = un;
            f = lanes(a0 + min(i + kWave + lane, n - 1), u, m);
            un = col[min(i + 2 * kWave + lane, n - 1)];
        }
        larcs += (unsigned)__popcll(xj);
        pairs += (unsigned)__popcll(bal);
        while (bal) take_matches(bal, xj, rj, 0, [&](unsigned long long v, int) { acc.add(v, sh); });
    }
    ac.larcs += larcs;
    if (lane == 0) {
        ac.pairs += pairs;
        ac.arcs += (unsigned)(a1 - a0);
    }
}

// Per-lane counters the path-count finalisation feeds.
struct SigCounters {
    unsigned edges = 0, full_n = 0, full_m = 0, lent = 0;
    unsigned long long act = 0, ovf = 0;
    int maxe = INT_MIN, mine = INT_MAX;
    ArcCounters ac;
};

// Store the path counts s of a new vertex (lanes m, row address ra).
template <int OP>
__device__ __forceinline__ void sig_store(const RowSum<OP> &s, unsigned long long m, unsigned long long ra,
                                          unsigned long long limit, unsigned long long &ovf, SigCounters &sc) {
    row_store(ra, row_slot(m), OP == OP_U64 ? s.lo : as_u64(s.d));
    if (OP == OP_U64) {
        // (lanes outside m hold a zero sum)
        ovf |= __ballot(s.hi != 0u || s.lo > limit);
    } else if (s.d > 0.0) {
        int ex;
        frexp(s.d, &ex);
        sc.maxe = max(sc.maxe, ex);
        sc.mine = min(sc.mine, ex);
    }
}

// Dependencies of one (vertex, lane) from the sum acc of its successors' c:
// delta, and c = (1 + delta) / sigma.
template <int MODE>
__device__ __forceinline__ void bwd_values(unsigned long long raw, double acc, int sh, int shn, double &delta,
                                           double &c) {
    const double sv = MODE ? ldexp(as_f64(raw), -sh) : (double)raw;
    delta = sv * acc;
    if (MODE) delta = ldexp(delta, -shn);
    c = (1.0 + delta) / sv;
}

// Packing of up to kBudget / 2 entries into one list of positions (arcs, or
// (entry, source) pairs), 64 positions to a chunk.  A bit per position marks
// where an entry starts; an entry's record is found by counting the starts up
// to a position: one broadcast read of the word and one read of the record per
// chunk (searching the prefix sums across lanes took six dependent LDS
// round trips and five more to fetch the entry's values).
constexpr int kPack = 64;                // entries of degree <= kPack are packed
constexpr int kPackEntries = kBudget * kMergeMax / 2;
constexpr int kPackWords = kPackEntries + 4;  // up to 64 positions per entry
struct Packing {
    unsigned long long start[kPackWords];
    uint4 rec[kPackEntries];
    uint4 rec2[kPackEntries];
};

__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Enter the packing: this lane's entry covers cnt positions (0: not packed)
// and has the records r and r2.  Returns the number of positions (uniform) and this
// entry's first one in off.
__device__ __forceinline__ int pack_entries(Packing &pk, int cnt, uint4 r, uint4 r2, int &off) {
    const int incl = wave_incl_scan(cnt);
    off = incl - cnt;
    const int total = __builtin_amdgcn_readlane(incl, 63);
    for (int i = lane_id(); i < (total + 63) / 64; i += kWave) pk.start[i] = 0ull;
    wave_lds_fence();
    const unsigned long long on = __ballot(cnt > 0);
    if (cnt > 0) {
        const int rank = (int)lanes_below(on);
        r.x -= (unsigned)off;  // arc of position i: r.x + i
        r2.z = (unsigned)off;
        pk.rec[rank] = r;
        pk.rec2[rank] = r2;
        atomicOr(&pk.start[off >> 6], 1ull << (off & 63));
    }
    wave_lds_fence();
    return total;
}
// Rank of the entry that holds position 64 * c + lane; before = entries that
// start before chunk c (advanced to the next chunk).
__device__ __forceinline__ int packed_rank(const Packing &pk, int c, int &before) {
    const unsigned long long w = readlane_u64(pk.start[c], 0);
    const int lane = lane_id();
    const int r = before + (int)lanes_below(w) + (int)((w >> lane) & 1ull) - 1;
    before += __popcll(w);
    return r;
}

// Index of the j-th set bit (j counted from 0) of m; m has more than j bits.
__device__ __forceinline__ int nth_set_bit(unsigned long long m, int j) {
    for (; j > 0; --j) m &= m - 1;
    return __ffsll(m) - 1;
}

// Sums of a group's packed entries: every entry's arcs in CSR order, 64 arcs
// of the list per chunk; fin(owner lane, sum) is called when an entry's last
// match has been added (an entry without matches is passed over).  Returns
// with the last entry's sum in acc and its lane in cur (-1: no match at all).
// Pipelined like row_arcs: what a chunk needs (record, column, frontier word)
// is requested one chunk ahead.
template <int OP, class Lanes, class Fin>
__device__ __forceinline__ void row_packed(const Packing &pk, int total, Lanes lanes, int sh,
                                           const int32_t *__restrict__ col, Slab slab, RowSum<OP> &acc,
                                           int &cur, ArcCounters &ac, Fin fin) {
    const int lane = lane_id();
    cur = -1;
    if (total == 0) return;
    int before = 0;
    unsigned larcs = 0, pairs = 0;
    // positions beyond the last one read the last entry's record and its last arc
    uint4 r = pk.rec[packed_rank(pk, 0, before)];
    int e = (int)r.x + min(lane, total - 1);
    int u = col[e];
    unsigned long long f = lanes(e, u, ((unsigned long long)r.z << 32) | r.y);
    int own = (int)r.w;
    uint4 rn = r;
    int un = u;
    if (kWave < total) {
        rn = pk.rec[packed_rank(pk, 1, before)];
        e = (int)rn.x + min(kWave + lane, total - 1);
        un = col[e];
    }
    for (int base = 0; base < total; base += kWave) {
        const unsigned long long xj = base + lane < total ? f : 0ull;
        const unsigned long long rj = slab.row(u);
        const int ownj = own;
        unsigned long long bal = __ballot(xj != 0ull);
        if (base + kWave < total) {
            u = un;
            own = (int)rn.w;
            f = lanes(e, u, ((unsigned long long)rn.z << 32) | rn.y);
            if (base + 2 * kWave < total) {
                rn = pk.rec[packed_rank(pk, base / kWave + 2, before)];
                e = (int)rn.x + min(base + 2 * kWave + lane, total - 1);
                un = col[e];
            }
        }
        larcs += (unsigned)__popcll(xj);
        pairs += (unsigned)__popcll(bal);
        while (bal) {
            take_matches(bal, xj, rj, ownj, [&](unsigned long long v, int o) {
                if (o != cur) {
                    if (cur >= 0) fin(cur, acc);
                    acc.clear();
                    cur = o;
                }
                acc.add(v, sh);
            });
        }
    }
    ac.larcs += larcs;
    if (lane == 0) {
        ac.pairs += pairs;
        ac.arcs += (unsigned)total;
    }
}

// Entry-lane items: when the entries of a group carry few sources each, the
// per-source sums run one thread per (entry, source) pair instead of one
// wavefront lane per source: each thread scans its entry's arcs [e0, e1)
// on its own and reads only source k's value of each matched far end.  Four
// arcs are followed at once (columns, then words, then values), and
// use(value) is called in CSR order, so the sum has the same bits as in the
// per-lane form.  Returns the matches.
template <class Use>
__device__ __forceinline__ unsigned item_arcs(const Tagged *fw, uint32_t T, int k, int e0, int e1,
                                              const int32_t *__restrict__ col, const unsigned long long *slab,
                                              Use use) {
    unsigned matched = 0;
    const int n = e1 - e0;
    for (int t = 0; t < n; t += 4) {
        int u[4];
        bool on[4];
        unsigned long long v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q] = col[e0 + min(t + q, n - 1)];
#pragma unroll
        for (int q = 0; q < 4; ++q) on[q] = t + q < n && tagged_lanes(fw, u[q], T, 1ull << k) != 0ull;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = on[q] ? slab[(size_t)u[q] * kLanes + k] : 0ull;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (on[q]) use(v[q]);
            matched += on[q] ? 1u : 0u;
        }
    }
    return matched;
}

// Finish the backward entries in `todo` (lanes of the group's entries: vertex
// v, live lanes M): their sums are parked in their delta rows, an entry that
// is not in `parked` had no match and sums to zero.  Four entries at a time, so
// that their path counts and sums are loaded together.
template <int MODE>
__device__ __forceinline__ void bwd_finish(unsigned long long todo, unsigned long long parked, unsigned long long M,
                                           int v, Slab sigma, Slab chat, Slab delta_slab, int sh, int shn) {
    while (todo) {
        unsigned long long raw[4], sum[4], mq[4];
        int vq[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int j = todo ? __ffsll(todo) - 1 : 0;
            mq[q] = todo ? readlane_u64(M, j) : 0ull;
            vq[q] = __builtin_amdgcn_readlane(v, j);
            todo &= todo - 1;
            raw[q] = row_load(sigma.row(vq[q]), row_slot(mq[q]));
            sum[q] = row_load(delta_slab.row(vq[q]), row_slot((parked >> j) & 1ull ? mq[q] : 0ull));
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned slot = row_slot(mq[q]);
            double delta, c;
            bwd_values<MODE>(raw[q], as_f64(sum[q]), sh, shn, delta, c);
            row_store(chat.row(vq[q]), slot, as_u64(c));
            row_store(delta_slab.row(vq[q]), slot, as_u64(delta));
            __builtin_amdgcn_sched_barrier(0);  // four divisions at once would not fit the registers
        }
    }
}

}  // namespace bcx
