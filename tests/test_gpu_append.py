"""Appends to a level queue around the size of a wavefront's staged run (224
entries are written at once, 288 fit) and of a workgroup's: levels of that
many vertices, with heavy vertices among them, in the per-source, batched and
weighted engines.  Scores against the oracle within 1e-10 (non-negative
terms)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


def _levels(k, heavy):
    """A root, k children, k grandchildren (one per child), and `heavy`
    vertices joined to every child and to a leaf fan of their own."""
    u = [np.zeros(k, int), np.arange(1, k + 1)]
    v = [np.arange(1, k + 1), np.arange(k + 1, 2 * k + 1)]
    n = 2 * k + 1
    for _ in range(heavy):
        u += [np.full(k, n), np.full(1100, n)]
        v += [np.arange(1, k + 1), np.arange(n + 1, n + 1101)]
        n += 1101
    return W.csr_from_edges(n, np.concatenate(u), np.concatenate(v))


@pytest.mark.parametrize("k,heavy", [(1, 1), (64, 0), (223, 0), (224, 2), (225, 0), (288, 1), (289, 0), (897, 3),
                                     (4097, 1)])
def test_runs(k, heavy):
    g = _levels(k, heavy)
    srcs = np.unique(np.concatenate([[0, 1, k, g.n - 1], np.random.default_rng(k).integers(0, g.n, 60)]))
    srcs = srcs.astype(np.int32)
    ref, _ = oracle.bc(g, srcs)
    say(f"[append] {k} children, {heavy} heavy, n={g.n}")
    with b.Graph(g) as G:
        for batch in (1, 64):
            for pol in (b.BC_POLICY_FORCE_PUSH_TPV, b.BC_POLICY_FORCE_PUSH_WPV, b.BC_POLICY_FORCE_PULL):
                G.run(srcs, batch=batch, policy=pol, flags=b.BC_RUN_ONE_QUEUE)
                assert_bc_close(G.scores(), ref)
        G.run(srcs, flags=b.BC_RUN_BLOCKS)
        assert_bc_close(G.scores(), ref)
    w = W.with_weights(g, 1, 3, seed=k)
    ref, _ = oracle.bc(w, srcs)
    with b.Graph(w) as G:
        G.run(srcs)
        assert_bc_close(G.scores(), ref)
