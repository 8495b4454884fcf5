"""Launch shapes: odd and even chunks of captured launches, launches without a
graph, one workgroup up to a full grid (steps that one workgroup runs alone and
steps that many share), and runs of one handle with changing numbers of
concurrent replicas.  Bits must not depend on any of it for one state machine;
across replica counts the sums are grouped differently (1e-13 relative)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 64])
@pytest.mark.parametrize("name", ["rmat", "grid", "grid_f64"])
def test_chunks_and_grids_same_bits(name, batch):
    g = W.rmat(11, 12, seed=3) if name == "rmat" else W.grid(40, 0.1, 0.002, seed=4)
    flags = b.BC_RUN_ONE_QUEUE | (b.BC_RUN_FORCE_F64 if name == "grid_f64" else 0)
    srcs = W.choose_sources(g, 20 if batch == 1 else 100, seed=5)
    ref, _ = oracle.bc(g, srcs)
    say(f"[launch] {name} batch={batch}")
    bits, levels = [], []
    with b.Graph(g) as G:
        for chunk, grid, more in ((0, 0, 0), (1, 1, 0), (3, 2, 0), (2, 31, 0), (5, 33, b.BC_RUN_NO_GRAPHS),
                                  (16, 64, b.BC_RUN_NO_GRAPHS), (1, 1536, 0)):
            G.run(srcs, batch=batch, flags=flags | more, chunk_steps=chunk, grid_blocks=grid)
            bits.append(G.scores())
            levels.append(G.level_stats())
    assert_bc_close(bits[0], ref)
    assert all(np.array_equal(bits[0], x) for x in bits)
    for lv in levels[1:]:
        assert np.array_equal(lv["entries"], levels[0]["entries"])
        assert np.array_equal(lv["visits"], levels[0]["visits"])


def test_changing_replica_counts_on_one_handle():
    g = W.rmat(13, 12, seed=8)
    srcs = W.choose_sources(g, 700, seed=9)
    ref, _ = oracle.bc(g, srcs)
    got = {}
    with b.Graph(g) as G:
        for r in (2, 8, 3, 0, 8, 1, 2):
            G.run(srcs, batch=64, replicas=r, flags=b.BC_RUN_NO_BLOCKS)
            s = G.scores()
            lv = G.level_stats()
            st = G.stats()
            assert int(lv["entries"].sum()) == st["queue_entries"] + len(srcs)  # level 0 holds the sources
            assert_bc_close(s, ref)
            assert r not in got or np.array_equal(got[r], s)
            got[r] = s
    for s in got.values():
        assert np.max(np.abs(s - got[1]) / np.maximum(got[1], 1e-300)) <= 1e-13
