"""Path-count and backward groups at the edges of their degree classes: the
64-arc packing (63, 64, 65 arcs), full chunks (127, 128, 129), one wavefront
against segments (1023, 1024, 1025), next to vertices of degree 1 and 2, for
one source and for full batches, under each way of summing light entries
(sources-per-entry threshold: never, always, default).  All ways must give the
same bits; scores against the oracle within 1e-10 (all terms non-negative: the
error is bounded by (levels + degree) * 2^-53, about 1e-13 here)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, check_detail, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


def _fan(degrees, seed, directed=False):
    """One centre per degree, joined to that many of a shared pool of
    vertices; the pool is a sparse random graph with a pendant tail."""
    rng = np.random.default_rng(seed)
    pool = max(degrees) + 40
    n = pool + len(degrees) + 3
    u, v = [], []
    for i, d in enumerate(degrees):
        far = rng.choice(pool, size=d, replace=False)
        u.append(np.full(d, pool + i))
        v.append(far)
    u.append(rng.integers(0, pool, 2 * pool)), v.append(rng.integers(0, pool, 2 * pool))
    tail = np.arange(n - 4, n - 1)
    u.append(tail), v.append(tail + 1)
    u, v = np.concatenate(u), np.concatenate(v)
    if directed:
        flip = rng.random(u.size) < 0.5
        u, v = np.where(flip, v, u), np.where(flip, u, v)
        return W.digraph_from_arcs(n, u, v)
    return W.csr_from_edges(n, u, v)


@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("degrees", [(1, 2, 31, 32, 33), (63, 64, 65, 66), (127, 128, 129, 130, 64, 64, 64),
                                     (1023, 1024, 1025, 1060, 2049)], ids=lambda d: "-".join(map(str, d)))
def test_degree_classes(degrees, directed):
    g = _fan(degrees, seed=len(degrees), directed=directed)
    rng = np.random.default_rng(7)
    srcs = rng.choice(g.n, size=min(130, g.n), replace=False).astype(np.int32)
    say(f"[degrees] {degrees} directed={directed} n={g.n} nnz={g.nnz}")
    with b.Graph(g) as G:
        for k in (1, 63, 64, 130):
            ref, _ = oracle.bc(g, srcs[:k])
            bits = []
            for il in (-1.0, 0.0, 65.0):
                for pol in (b.BC_POLICY_HEURISTIC, b.BC_POLICY_FORCE_PUSH_TPV, b.BC_POLICY_FORCE_PUSH_WPV,
                            b.BC_POLICY_FORCE_PULL):
                    for flags in (0, b.BC_RUN_FORCE_F64):
                        G.run(srcs[:k], batch=64, lanes_per_entry=il, policy=pol, flags=flags | b.BC_RUN_ONE_QUEUE)
                        got = G.scores()
                        assert_bc_close(got, ref)
                        if not flags:
                            bits.append(got)
            assert all(np.array_equal(bits[0], x) for x in bits)
        for i in (0, 5):
            check_detail(g, G.detail(srcs[:64], i, batch=64), srcs[i])
