"""When a run of the batched engine goes to the block engine by default, and
what it then depends on.  Scores against the oracle within 1e-10 relative
(non-negative terms)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


def _union(count, n=700):
    # about 8 n arcs a graph: one batch more than four for every 4,096
    return W.union([W.barabasi_albert(n + 7 * i, 4, seed=900 + i) for i in range(count)])


def _bits(G):
    return G.scores().view(np.uint64).copy()


@pytest.mark.parametrize("count,each,block", [(12, 1, True), (12, 70, True), (4, 60, False), (4, 65, True), (3, 60, False)])
def test_a_graph_s_last_sources_are_a_batch(count, each, block):
    # (5 batches are asked for: 12 graphs with one source have 12, 4 graphs with
    # 60 have 4, with 65 they have 8)
    u = _union(count)
    assert 4096 <= max(np.diff(u.row_ptr[u.vtx_offsets])) < 8192
    srcs = np.concatenate([np.arange(o, o + each) for o in u.vtx_offsets[:-1]]).astype(np.int32)
    ref, _ = oracle.bc(u, srcs)
    with b.Graph(u) as G:
        G.run(srcs)
        st = G.stats()
        say(f"[block choice] {count} graphs, {each} each: workgroups {st['block_workgroups']}")
        assert (st["block_workgroups"] > 0) == block
        assert_bc_close(G.scores(), ref)
        G.run(None, batch=64)  # every vertex: 12 batches a graph
        assert G.stats()["block_workgroups"] > 0
        with pytest.raises(b.BCError):
            G.run(np.array([0, u.n], np.int32))
        with pytest.raises(b.BCError):
            G.run(np.array([-1, 0], np.int32))


@pytest.mark.parametrize("graphs", [1, 5])
def test_a_run_that_exceeds_the_capacities_goes_on_as_usual(graphs):
    # a path of 6,000 vertices has more levels than a workgroup holds: the run
    # ends on the concurrent state machines that it would have had without the
    # block engine (same bits), and the block engine's memory is given back
    one = W.csr_from_edges(6000, np.arange(5999), np.arange(1, 6000))
    u = one if graphs == 1 else W.union([one] * graphs)
    srcs = np.concatenate([np.linspace(o, o + 5999, 640 // graphs) for o in range(0, u.n, 6000)]).astype(np.int32)
    ref, _ = oracle.bc(u, srcs)
    with b.Graph(u) as G:
        G.run(srcs, batch=64, flags=b.BC_RUN_NO_BLOCKS)
        want, st0, held = _bits(G), G.stats(), G.info()["device_bytes"]
        G.run(srcs, batch=64, flags=b.BC_RUN_BLOCKS)
        st = G.stats()
        say(f"[block choice] {graphs} paths: {st0['ms']:.0f} ms without, {st['ms']:.0f} ms after the block engine's pass")
        assert st["block_workgroups"] == 0 and st["grid_blocks"] == st0["grid_blocks"]
        assert st["n_batches"] == st0["n_batches"] and st["steps"] == st0["steps"]
        assert np.array_equal(_bits(G), want)
        assert_bc_close(G.scores(), ref)
        assert G.info()["device_bytes"] <= held + (1 << 20)
        G.run(srcs[:320], batch=64, flags=b.BC_RUN_BLOCKS)
        G.run(srcs[320:], batch=64, flags=b.BC_RUN_BLOCKS | b.BC_RUN_ACCUMULATE)
        assert_bc_close(G.scores(), ref)


def _smallest(u, srcs, lo, hi, ok, **opts):
    """Smallest cap (bytes above the handle's own, to 64 KiB) with which a new handle's run is `ok`."""
    def test(x):
        with b.Graph(u) as G:
            G.set_device_limit(G.info()["device_bytes"] + x)
            try:
                G.run(srcs, **opts)
            except b.BCError as e:
                assert e.status == 3
                return False
            return ok(G.stats())
    assert test(hi) and not test(lo)
    while hi - lo > 65536:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if test(mid) else (mid, hi)
    return hi


def test_engines_give_way_to_each_other_under_a_cap():
    # a cap under which each engine runs alone: they run in any order, and the
    # handle never holds more than the cap (parts of a union included)
    u = _union(12, 3000)
    srcs = np.concatenate([np.arange(o, o + 40) for o in u.vtx_offsets[:-1]]).astype(np.int32)
    ref, _ = oracle.bc(u, srcs)
    runs = {"block": dict(batch=64, flags=b.BC_RUN_BLOCKS), "general": dict(batch=64, flags=b.BC_RUN_NO_BLOCKS),
            "per source": dict(batch=1)}
    cap = _smallest(u, srcs, 0, 4 << 30, lambda st: st["block_workgroups"] > 0, **runs["block"])
    cap = max(cap, _smallest(u, srcs, 0, 4 << 30, lambda st: True, **runs["general"]))
    cap += 2 << 20  # the per-source state beside the general engine's
    say(f"[block choice] cap {cap >> 20} MiB above the handle")
    for top in (cap, cap + (256 << 20), cap + (1 << 30)):
        with b.Graph(u) as G:
            floor = G.info()["device_bytes"]
            G.set_device_limit(floor + top)
            for what in ("block", "general", "block", "per source", "general", "block"):
                G.run(srcs, **runs[what])
                st = G.stats()
                say(f"  {what}: workgroups {st['block_workgroups']}, {(G.info()['device_bytes'] - floor) >> 20} MiB")
                assert G.info()["device_bytes"] <= floor + top
                if what != "block":
                    assert st["block_workgroups"] == 0
                assert_bc_close(G.scores(), ref)


def test_overflowed_sources_find_room_under_a_cap():
    # the FP64 pass after the block engine's 64-bit pass takes the general engine
    u = W.union([W.barabasi_albert(900, 4, seed=31), W.grid(60, 0.05, 0.0, seed=21), W.barabasi_albert(1500, 4, seed=32)])
    srcs = np.arange(0, u.n, 7, dtype=np.int32)
    ref, modes = oracle.bc(u, srcs)
    assert modes.any()
    opts = dict(batch=64, flags=b.BC_RUN_BLOCKS)
    general = _smallest(u, srcs, 0, 2 << 30, lambda st: True, batch=64, flags=b.BC_RUN_NO_BLOCKS)
    for extra in (0, 2 << 20, 16 << 20, 64 << 20):
        with b.Graph(u) as G:
            floor = G.info()["device_bytes"]
            G.set_device_limit(floor + general + extra)
            G.run(srcs, **opts)
            st = G.stats()
            say(f"[block choice] {extra >> 20} MiB more: workgroups {st['block_workgroups']}, f64 {st['f64_sources']}")
            assert st["f64_sources"] == int(modes.sum())
            assert G.info()["device_bytes"] <= floor + general + extra
            assert_bc_close(G.scores(), ref)


def test_bits_do_not_depend_on_the_memory_that_is_left():
    # lanes and chunks follow from the sizes; a cap only takes workgroups away
    u = _union(12, 3000)
    srcs = np.concatenate([np.arange(o, o + 200) for o in u.vtx_offsets[:-1]]).astype(np.int32)
    ref, _ = oracle.bc(u, srcs)
    opts = dict(flags=b.BC_RUN_BLOCKS)
    with b.Graph(u) as G:
        G.run(srcs, **opts)
        st0, want = G.stats(), _bits(G)
        assert_bc_close(G.scores(), ref)
    # (lists of the run included: about 12 MiB of partial scores)
    need = _smallest(u, srcs, 0, 4 << 30, lambda st: st["block_workgroups"] > 0, **opts)
    for extra in (0, 40 << 20, 400 << 20):
        with b.Graph(u) as G:
            floor = G.info()["device_bytes"]
            G.set_device_limit(floor + need + extra)
            G.run(srcs, **opts)
            st = G.stats()
            say(f"[block choice] {(need + extra) >> 20} MiB: workgroups {st['block_workgroups']} of {st0['block_workgroups']}")
            assert 0 < st["block_workgroups"] < st0["block_workgroups"]
            assert st["n_batches"] == st0["n_batches"] and st["block_chunks"] == st0["block_chunks"]
            assert np.array_equal(_bits(G), want)
            assert G.info()["device_bytes"] <= floor + need + extra


def test_default_needs_half_of_the_workgroups():
    u = _union(12, 3000)
    srcs = np.concatenate([np.arange(o, o + 200) for o in u.vtx_offsets[:-1]]).astype(np.int32)
    ref, _ = oracle.bc(u, srcs)
    with b.Graph(u) as G:
        G.run(srcs)
        full = G.stats()["block_workgroups"]
        held = G.info()["device_bytes"]
    for share, block in ((0.3, False), (0.9, True)):
        with b.Graph(u) as G:
            floor = G.info()["device_bytes"]
            cap = int((held - floor) * share)
            G.set_device_limit(floor + cap)
            for _ in range(2):
                G.run(srcs)
                st = G.stats()
                say(f"[block choice] {share} of {(held - floor) >> 20} MiB: workgroups {st['block_workgroups']} of {full}, {st['ms']:.2f} ms")
                assert (st["block_workgroups"] > 0) == block
                assert G.info()["device_bytes"] <= floor + cap
                assert_bc_close(G.scores(), ref)


def _caterpillar(spine, leaves):
    """A path whose vertices have `leaves` leaves each."""
    s = np.arange(spine)
    u = np.concatenate([s[:-1], np.repeat(s, leaves)])
    v = np.concatenate([s[1:], np.arange(spine, spine * (1 + leaves))])
    return W.csr_from_edges(spine * (1 + leaves), u, v)


def _strip(rows, cols):
    ids = np.arange(rows * cols).reshape(cols, rows)  # (numbered across: local)
    u = np.concatenate([ids[:, :-1].ravel(), ids[:-1].ravel()])
    v = np.concatenate([ids[:, 1:].ravel(), ids[1:].ravel()])
    return W.csr_from_edges(rows * cols, u, v)


def _star_and_cycles(n):
    """A star, and a cycle of `n` vertices beside it."""
    c = np.arange(n)
    return W.csr_from_edges(n + 100, np.concatenate([c, np.full(99, n)]),
                            np.concatenate([np.roll(c, -1), np.arange(n + 1, n + 100)]))


LEVELS = {
    # large and thin: a vertex is on as many levels as a batch has sources (32 and 64)
    "caterpillars, 32": (lambda: W.union([_caterpillar(3000, 9)] * 4), 1500, 0, True),
    "caterpillars, 64": (lambda: W.union([_caterpillar(3000, 9)] * 4), 2900, 0, True),
    "caterpillars, 64, kept": (lambda: W.union([_caterpillar(3000, 9)] * 4), 2900, b.BC_KEEP_ORDER, True),
    "strips": (lambda: W.union([_strip(4, 4500 + i) for i in range(4)]), 560, 0, False),  # more than 4,096 levels
    # as large, few levels
    "preferential": (lambda: W.union([W.barabasi_albert(18000 + 500 * i, 4, seed=i) for i in range(8)]), 420, 0, True),
    "preferential, kept": (lambda: W.union([W.barabasi_albert(18000 + 500 * i, 4, seed=i) for i in range(8)]), 420,
                           b.BC_KEEP_ORDER, True),
    "path 4000": (lambda: _strip(1, 4000), 700, 0, True),
    "path 6000": (lambda: _strip(1, 6000), 700, 0, False),  # 6,000 levels, 4,096 fit
    "path 6000, kept": (lambda: _strip(1, 6000), 700, b.BC_KEEP_ORDER, False),
    "strip 2 x 4000": (lambda: _strip(2, 4000), 900, 0, True),
    "strip 2 x 4100": (lambda: _strip(2, 4100), 900, 0, False),
    "star, cycle 8000": (lambda: _star_and_cycles(8000), 700, 0, True),
    "star, cycle 8300": (lambda: _star_and_cycles(8300), 700, 0, False),
}


@pytest.mark.parametrize("name", LEVELS)
def test_default_keeps_to_a_workgroup_s_queue_and_levels(name):
    # a run is never tried on the block engine only to be given up: where it is not
    # taken, the handle holds no more than one that was told not to use it
    make, each, flags, block = LEVELS[name]
    u = make()
    off = u.vtx_offsets if getattr(u, "vtx_offsets", None) is not None and len(u.vtx_offsets) > 2 else [0, u.n]
    rng = np.random.default_rng(1)
    srcs = np.concatenate([np.sort(rng.permutation(min(o1 - o0, 3000 if "cat" in name else o1 - o0))[:each]) + o0
                           for o0, o1 in zip(off[:-1], off[1:])]).astype(np.int32)
    seen = []
    for opts in ({}, {"flags": b.BC_RUN_NO_BLOCKS})[: 1 if block else 2]:
        with b.Graph(u, flags=flags) as G:
            G.run(srcs, **opts)
            st = G.stats()
            seen.append((G.info()["device_bytes"], hash(_bits(G).tobytes())))
            say(f"[block choice] {name} {opts}: workgroups {st['block_workgroups']}, {st['ms']:.1f} ms, {seen[-1][0] >> 20} MiB")
            assert (st["block_workgroups"] > 0) == block
    assert len(set(seen)) == 1
    with b.Graph(u, flags=flags) as G:  # and against the oracle, over fewer sources
        few = srcs[:: max(1, len(srcs) // 24)]
        G.run(few, flags=b.BC_RUN_BLOCKS)
        assert_bc_close(G.scores(), oracle.bc_sliced(u, few, threads=8)[0])


def test_memory_that_is_held_stays_in_use():
    # graphs of 60,000 vertices take some 100 MB a workgroup; with the rest of the
    # device memory taken after the first run, the second has what it needs
    import torch

    u = W.union([W.barabasi_albert(60000, 3, seed=40 + i) for i in range(4)])
    srcs = np.concatenate([np.arange(o, o + 2048) for o in u.vtx_offsets[:-1]]).astype(np.int32)
    with b.Graph(u) as G:
        before = G.info()["device_bytes"]
        G.run(srcs, batch=64)
        st0, want, held = G.stats(), _bits(G), G.info()["device_bytes"]
        assert st0["block_workgroups"] == 128
        left = (held - before) // 5  # (three quarters of 1.2 times would be too little)
        take = torch.cuda.mem_get_info()[0] - left
        say(f"[block choice] {(held - before) >> 20} MiB held, {take >> 20} MiB taken, {left >> 20} MiB left")
        assert left >= 2 << 30 and take > 0
        rest = torch.empty(take, dtype=torch.uint8, device="cuda")
        try:
            G.run(srcs, batch=64)
        finally:
            del rest
            torch.cuda.empty_cache()
        st = G.stats()
        say(f"[block choice] workgroups {st['block_workgroups']}, {st['ms']:.1f} ms after {st0['ms']:.1f} ms")
        assert st["block_workgroups"] == st0["block_workgroups"]
        assert np.array_equal(_bits(G), want) and G.info()["device_bytes"] == held
