"""Concurrent state machines of a single graph under a device-memory cap: a
list that asks for more of them than fit takes one, and lists that ask for
fewer keep theirs.  Scores against the oracle within 1e-10 relative."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(G, srcs, **opts):
    G.run(srcs, batch=8, flags=b.BC_RUN_NO_BLOCKS, **opts)
    return G.scores().view(np.uint64).copy()


@pytest.mark.parametrize("first", ["short", "long"])
def test_a_longer_list_does_not_cost_a_shorter_one_its_machines(first):
    # 40 batches ask for 4 machines, 64 for 8
    g = W.rmat(11, 16, seed=31)
    lists = {"short": W.choose_sources(g, 320, seed=7), "long": W.choose_sources(g, 512, seed=8)}
    ref = {k: oracle.bc(g, s)[0] for k, s in lists.items()}
    want = {}
    with b.Graph(g) as G:
        floor = G.info()["device_bytes"]
        want["short"] = _run(G, lists["short"])
        four = G.info()["device_bytes"] - floor
        machine = G.stats()["grid_blocks"]
        _run(G, lists["long"])
        assert G.info()["device_bytes"] - floor > 1.9 * four  # 8 machines
    with b.Graph(g) as G:
        want["long"] = _run(G, lists["long"], replicas=1)
        assert G.stats()["grid_blocks"] != machine
    with b.Graph(g) as G:
        G.set_device_limit(floor + int(1.6 * four))
        for what in (first, "short", "long", "short"):
            got = _run(G, lists[what])
            say(f"[replica cap] {what}: {(G.info()['device_bytes'] - floor) >> 10} KiB of {int(1.6 * four) >> 10}")
            assert np.array_equal(got, want[what])
            assert (G.stats()["grid_blocks"] == machine) == (what == "short")
            assert_bc_close(G.scores(), ref[what])
            assert G.info()["device_bytes"] <= floor + int(1.6 * four)
        G.set_device_limit(0)
        _run(G, lists["long"])  # decided again
        assert G.stats()["grid_blocks"] == machine


def test_the_handle_s_own_machine_counts_beside_its_parts():
    g = W.rmat(11, 16, seed=31)
    srcs = W.choose_sources(g, 320, seed=7)
    ref, _ = oracle.bc(g, srcs)
    with b.Graph(g) as G:
        floor = G.info()["device_bytes"]
        _run(G, srcs)
        cap = floor + int(1.05 * (G.info()["device_bytes"] - floor))  # the parts, and not the handle's own beside them
        G.set_device_limit(cap)
        for opts in ({}, {"replicas": 1}, {}, {"replicas": 1}):
            _run(G, srcs, **opts)
            say(f"[replica cap] {opts}: {(G.info()['device_bytes'] - floor) >> 10} of {(cap - floor) >> 10} KiB")
            assert G.info()["device_bytes"] <= cap
            assert_bc_close(G.scores(), ref)


def test_more_machines_than_usual_are_given_back():
    # 16 while they are asked for, then as many as a handle that never had them
    g = W.rmat(11, 16, seed=31)
    short, long = W.choose_sources(g, 320, seed=7), W.choose_sources(g, 512, seed=8)
    with b.Graph(g) as G:
        _run(G, long)
        want, usual = _run(G, short), G.info()["device_bytes"]  # 8, of which a short list uses 4
    with b.Graph(g) as G:
        _run(G, long, replicas=16)
        most = G.info()["device_bytes"]
        assert most > 1.8 * usual
        _run(G, long, replicas=16)
        assert G.info()["device_bytes"] == most
        assert np.array_equal(_run(G, short), want)
        assert G.info()["device_bytes"] <= usual + (1 << 20)
        _run(G, long)
        assert np.array_equal(_run(G, short), want)
        assert G.info()["device_bytes"] <= usual + (1 << 20)
