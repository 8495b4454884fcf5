"""Weighted graphs under a device-memory cap.  What runs under a cap depends on
the cap alone: a list that runs under one runs under every larger one, and
after any other run on the same handle (the engines' states and the lists of
earlier runs give way).  Scores against the oracle within 1e-10 relative
(non-negative terms); the handle never holds more than the cap."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


def _graph(scale):
    base = W.rmat(scale, 16, seed=65)
    return W.with_weights(base, 1, 50, seed=9), base


def _runs(G, srcs, **opts):
    """Engine of the run: 'wide', 'workgroups', or None where it is refused."""
    try:
        G.run(srcs, **opts)
    except b.BCError as e:
        assert e.status == 3
        return None
    return "wide" if G.stats()["n_batches"] else "workgroups"


def _smallest(g, srcs, want, lo, hi, **opts):
    """Smallest cap (bytes above the handle's own, to 4 KiB) with which a new handle's run takes an engine of `want`."""
    def ok(x):
        with b.Graph(g) as G:
            G.set_device_limit(G.info()["device_bytes"] + x)
            return _runs(G, srcs, **opts) in want
    assert ok(hi) and not ok(lo)
    while hi - lo > 4096:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if ok(mid) else (mid, hi)
    return hi


@pytest.mark.parametrize("lanes", [0, 1, 16])
def test_every_larger_cap_runs(lanes):
    g, base = _graph(11)
    srcs = W.choose_sources(base, 60, seed=10)
    ref, _ = oracle.bc(g, srcs)
    seen = []
    with b.Graph(g) as H:
        floor = H.info()["device_bytes"]
        for x in range(64 << 10, 12 << 20, 192 << 10):
            with b.Graph(g) as G:
                G.set_device_limit(floor + x)
                how = _runs(G, srcs, weighted_lanes=lanes)
                assert G.info()["device_bytes"] <= floor + x
                if how:
                    assert_bc_close(G.scores(), ref)
            # and a handle that has run under every smaller cap
            H.set_device_limit(floor + x)
            assert _runs(H, srcs, weighted_lanes=lanes) == how
            assert H.info()["device_bytes"] <= floor + x
            assert how or not any(seen), f"refused {x} bytes above the handle, a smaller cap ran"
            seen.append(how)
    say(f"[weighted memory] lanes {lanes}: {[(h, seen.count(h)) for h in dict.fromkeys(seen)]}")
    assert seen[0] is None and seen[-1]
    assert lanes or {"workgroups", "wide"} <= set(seen)


@pytest.mark.parametrize("other", [1, 16])
def test_engines_give_way_to_each_other(other):
    g, base = _graph(12)
    srcs = W.choose_sources(base, 60, seed=10)
    ref, _ = oracle.bc(g, srcs)
    top = 64 << 20
    cap = max(_smallest(g, srcs, ("wide",), 0, top),
              _smallest(g, srcs, ("workgroups",), 0, top, weighted_lanes=other))
    say(f"[weighted memory] both alone from {cap} bytes")
    with b.Graph(g) as G:
        G.set_device_limit(G.info()["device_bytes"] + cap)
        bits = None
        for _ in range(2):
            assert _runs(G, srcs) == "wide"
            assert_bc_close(G.scores(), ref)
            bits = G.scores().view(np.uint64).copy() if bits is None else bits
            assert np.array_equal(G.scores().view(np.uint64), bits)
            assert _runs(G, srcs, weighted_lanes=other) == "workgroups"
            assert_bc_close(G.scores(), ref)


def test_longer_list_beside_the_wide_state():
    # the wide state fits with the lists of 64 sources and not with those of 1000
    g, base = _graph(14)
    srcs = W.choose_sources(base, 1000, seed=10)
    cap = _smallest(g, srcs[:64], ("wide",), 0, 256 << 20)
    ref, _ = oracle.bc_sliced(g, srcs, threads=8)
    with b.Graph(g) as G:
        G.run(srcs)
        assert G.stats()["n_batches"] == 16  # without a cap both lists take the wide engine
    with b.Graph(g) as G:
        G.set_device_limit(G.info()["device_bytes"] + cap)
        assert _runs(G, srcs[:64]) == "wide"
        assert _runs(G, srcs) == "workgroups"
        assert_bc_close(G.scores(), ref)
        assert _runs(G, srcs[:64]) == "wide"


def test_alternating_widths_keep_their_memory():
    # one source and 16 per workgroup in turn, asked for and chosen by the
    # length of the list (1 up to 2,560 sources on this path, 16 beyond)
    base = W.csr_from_edges(600, np.arange(599), np.arange(1, 600))
    g = W.with_weights(base, 1, 9, seed=5)
    rng = np.random.default_rng(3)
    short, long = (rng.integers(0, g.n, k).astype(np.int32) for k in (40, 2700))
    refs = [oracle.bc(g, s)[0] for s in (short, long)]
    with b.Graph(g) as G:
        held = []
        for r in range(3):
            for s, ref in zip((short, long), refs):
                for lanes in (0, 1, 16):
                    G.run(s, weighted_lanes=lanes)
                    assert_bc_close(G.scores(), ref)
                    held.append(G.info()["device_bytes"])
    say(f"[weighted memory] device bytes run by run {held}")
    assert len(set(held[6:])) == 1
