"""Segments of heavy vertices, whose length follows the graph's arcs (128 below
2^20 arcs, then 512 and 1,024; weighted graphs 128, 256 and 512): vertices with
one arc less, as many and one more than each length and its double, in graphs
of every class.  d and path counts exact, scores against the oracle within
1e-10 (non-negative terms)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, check_detail, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu

DEGREES = [d + e for d in (128, 256, 512, 1024, 2048) for e in (-1, 0, 1)]


def _graph(arcs):
    rng = np.random.default_rng(arcs)
    n = max(arcs // 8, 5000)
    u = [rng.integers(0, n, arcs // 2)]
    v = [rng.integers(0, n, arcs // 2)]
    for i, d in enumerate(DEGREES):
        u.append(np.full(d, n + i))
        v.append(rng.choice(5000, size=d, replace=False))
    return W.csr_from_edges(n + len(DEGREES), np.concatenate(u), np.concatenate(v))


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("arcs", [40_000, 1_200_000, 6_500_000])
def test_segment_lengths(arcs, weighted):
    g = _graph(arcs)
    if weighted:
        g = W.with_weights(g, 1, 3, seed=1)
    rng = np.random.default_rng(3)
    srcs = np.concatenate([[g.n - 1, g.n - 5], rng.integers(0, g.n, 2 if arcs > 2_000_000 else 66)]).astype(np.int32)
    ref, _ = oracle.bc(g, srcs)
    say(f"[segments] {g.nnz} arcs, weighted={weighted}")
    with b.Graph(g) as G:
        pols = (b.BC_POLICY_HEURISTIC,) if weighted else (b.BC_POLICY_FORCE_PUSH_TPV, b.BC_POLICY_FORCE_PUSH_WPV,
                                                          b.BC_POLICY_FORCE_PULL)
        for pol in pols:
            G.run(srcs, batch=0 if weighted else 64, policy=pol)
            assert_bc_close(G.scores(), ref)
        if not weighted:
            check_detail(g, G.detail(srcs, dump_index=0, batch=64), int(srcs[0]))
