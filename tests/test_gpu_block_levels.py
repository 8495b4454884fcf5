"""Per-level records of runs on the block engine: whole numbers, so they add up
to the run's statistics, and with batches of the same width (sources of a batch
reach the same vertices on the same levels) visits and entries are the
general engine's."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


def _cases():
    path = W.csr_from_edges(900, np.arange(899), np.arange(1, 900))  # beyond the levels kept per workgroup
    return {"er": W.erdos_renyi(1500, 8.0, seed=3), "path": path, "rmat": W.rmat(11, 16, seed=4),
            "union": W.union([W.barabasi_albert(400 + 50 * i, 3, seed=i) for i in range(9)] + [path])}


@pytest.mark.parametrize("name", ["er", "path", "rmat", "union"])
def test_level_records_of_the_block_engine(name):
    g = _cases()[name]
    srcs = np.sort(np.random.default_rng(5).permutation(g.n)[:600]).astype(np.int32)
    say(f"[block levels] {name}")
    with b.Graph(g) as G:
        G.run(srcs, batch=16, flags=b.BC_RUN_NO_BLOCKS)
        want = G.level_stats()
        for opts in ({"batch": 16, "flags": b.BC_RUN_BLOCKS}, {"flags": b.BC_RUN_BLOCKS}):
            G.run(srcs, **opts)
            st, lv = G.stats(), G.level_stats()
            assert st["block_workgroups"] > 0
            assert len(lv["visits"]) == st["max_levels"]
            assert int(lv["visits"].sum()) == st["forward_levels"]
            assert int(lv["visits"][0]) == st["n_batches"]
            assert int(lv["entries"][1:].sum()) == st["queue_entries"]
            assert lv["variant"].sum(axis=0).tolist() == st["variant_levels"]
            assert int(lv["arcs"].sum()) == st["arcs_scanned"]
            assert (lv["ms"] >= 0).all() and lv["ms"].sum() > 0
            if opts.get("batch"):
                assert np.array_equal(lv["visits"], want["visits"])
                assert np.array_equal(lv["entries"], want["entries"])


def test_records_after_a_pass_that_was_given_up():
    # a path of 6,000 vertices leaves the block engine: its records are not counted
    g = W.csr_from_edges(6000, np.arange(5999), np.arange(1, 6000))
    srcs = np.linspace(0, 5999, 96).astype(np.int32)
    with b.Graph(g) as G:
        G.run(srcs, batch=64, flags=b.BC_RUN_NO_BLOCKS)
        want = G.level_stats()
        G.run(srcs, batch=64, flags=b.BC_RUN_BLOCKS)
        got = G.level_stats()
    assert np.array_equal(got["visits"], want["visits"]) and np.array_equal(got["entries"], want["entries"])


@pytest.mark.parametrize("ns,flags,batch,used", [
    (600, b.BC_RUN_BLOCKS, 0, 8), (2100, b.BC_RUN_BLOCKS, 0, 16), (600, b.BC_RUN_BLOCKS, 32, 32),
    (600, b.BC_RUN_NO_BLOCKS, 0, 64), (600, b.BC_RUN_NO_BLOCKS, 16, 16), (600, b.BC_RUN_NO_BLOCKS | b.BC_RUN_ONE_QUEUE, 8, 8),
    (20, 0, 1, 1)])
def test_statistics_name_the_width_that_was_used(ns, flags, batch, used):
    g = W.erdos_renyi(1500, 8.0, seed=3)
    srcs = np.random.default_rng(5).integers(0, g.n, ns).astype(np.int32)
    with b.Graph(g) as G:
        G.run(srcs, batch=batch, flags=flags)
        st = G.stats()
        assert st["batch"] == used
        if used > 1:
            assert st["n_batches"] == -(-ns // used)
