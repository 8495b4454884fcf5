"""The block engine's own choices: the lanes of a batch when the caller leaves
them open, and when a run goes to it by default.  Scores are checked against
the oracle within the 1e-10 relative that every 64-bit run keeps; the choice
must not depend on anything but the sizes, so a repeated run has the same
bits."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


# sources: one under, at and over the batches of 8, 16 and 32 lanes that an
# MI355X's 256 workgroups hold, the last ones past every step of the choice
@pytest.mark.parametrize("ns,K", [(9, 8), (2048, 8), (2049, 16), (4097, 32), (8193, 64)])
def test_lanes_left_open(ns, K):
    g = W.erdos_renyi(1200, 6.0, seed=5)
    rng = np.random.default_rng(ns)
    srcs = rng.integers(0, g.n, ns).astype(np.int32)
    ref, _ = oracle.bc(g, srcs)
    with b.Graph(g) as G:
        G.run(srcs, flags=b.BC_RUN_BLOCKS)
        st = G.stats()
        got = G.scores().copy()
        say(f"[block lanes] {ns} sources: batches {st['n_batches']} workgroups {st['block_workgroups']}")
        assert st["block_workgroups"] > 0
        assert st["n_batches"] == -(-ns // K)
        assert_bc_close(got, ref)
        G.run(srcs, flags=b.BC_RUN_BLOCKS)
        assert np.array_equal(G.scores().view(np.uint64), got.view(np.uint64))


@pytest.mark.parametrize("batches,block", [(8, False), (40, True)])
def test_default_follows_the_arcs(batches, block):
    # R-MAT of 2^12 vertices has about 110,000 arcs: 4 batches and one per
    # 4,096 of them (about 30 in all) and more go to the block engine
    g = W.rmat(12, 16, seed=3)
    assert 8 * 4096 < g.nnz < 35 * 4096
    srcs = np.random.default_rng(2).permutation(g.n).astype(np.int32)[: batches * 64]
    ref, _ = oracle.bc_sliced(g, srcs, threads=8)
    with b.Graph(g) as G:
        G.run(srcs)
        assert (G.stats()["block_workgroups"] > 0) == block
        assert_bc_close(G.scores(), ref)
