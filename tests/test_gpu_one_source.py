"""The per-source engine at the edges of its lane groups: 8 lanes with four
arcs each up to 64 arcs, a wavefront up to 512, segments beyond; vertices of
every class next to each other, levels that do not fill a wavefront's eight
entries, and unvisited vertices spread over a pull level's runs.  Scores
against the oracle within 1e-10 (all terms non-negative: the error is bounded
by (levels + degree) * 2^-53), the same bits run to run."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, check_detail, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


def _hubs(degrees, n, seed):
    rng = np.random.default_rng(seed)
    u = [rng.integers(0, n, n)]
    v = [rng.integers(0, n, n)]
    for i, d in enumerate(degrees):
        u.append(np.full(d, n + i))
        v.append(rng.choice(n, size=d, replace=False))
    m = n + len(degrees)
    return W.csr_from_edges(m, np.concatenate(u), np.concatenate(v))


@pytest.mark.parametrize("degrees,n", [((1, 7, 8, 9), 33), ((31, 32, 33, 63), 127), ((64, 65, 66, 128, 129), 500),
                                       ((511, 512, 513, 600), 700), ((256, 257, 1024, 1025, 1537), 2049)],
                         ids=lambda x: "-".join(map(str, x)) if isinstance(x, tuple) else str(x))
def test_lane_groups(degrees, n):
    g = _hubs(degrees, n, seed=n)
    srcs = np.random.default_rng(1).choice(g.n, size=9, replace=False).astype(np.int32)
    srcs[0] = g.n - 1  # a hub as the source
    ref, _ = oracle.bc(g, srcs)
    say(f"[one source] degrees {degrees} n={g.n}")
    with b.Graph(g) as G:
        for pol in (b.BC_POLICY_HEURISTIC, b.BC_POLICY_FORCE_PUSH_TPV, b.BC_POLICY_FORCE_PUSH_WPV,
                    b.BC_POLICY_FORCE_PULL):
            for flags in (0, b.BC_RUN_FORCE_F64):
                bits = []
                for _ in range(2):
                    G.run(srcs, batch=1, policy=pol, flags=flags)
                    bits.append(G.scores().view(np.uint64).copy())
                assert np.array_equal(bits[0], bits[1])
                assert_bc_close(G.scores(), ref)
        det = G.detail(srcs, dump_index=0, batch=1)
        check_detail(g, det, int(srcs[0]))


def test_segment_sums_past_64_bits():
    # counts beyond the limit in an eight-lane group, a wavefront and a
    # segment: the source is flagged and runs again in FP64
    g = _hubs((40, 300, 900), 1200, seed=3)
    srcs = np.arange(6, dtype=np.int32)
    ref, _ = oracle.bc(g, srcs)
    with b.Graph(g) as G:
        for pol in (b.BC_POLICY_FORCE_PUSH_TPV, b.BC_POLICY_FORCE_PULL):
            G.run(srcs, batch=1, policy=pol, sigma_limit=2)
            assert G.stats()["f64_sources"] == len(srcs)
            assert_bc_close(G.scores(), ref)
