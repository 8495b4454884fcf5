"""The engine a weighted run takes when weighted_lanes is left open: lists
around the sizes where it changes, on graphs on either side of the line
between a source per workgroup and the whole GPU per batch.  Scores against
the oracle within 1e-10 (non-negative terms), run to run the same bits."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, check_detail, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns", [1, 64, 65, 512, 2560, 2561])
@pytest.mark.parametrize("name", ["path", "grid", "rmat9", "directed"])
def test_list_sizes(name, ns):
    g = {"path": lambda: W.csr_from_edges(120, np.arange(119), np.arange(1, 120)),
         "grid": lambda: W.grid(18, 0.1, 0.01, seed=2), "rmat9": lambda: W.rmat(9, 8, seed=2),
         "directed": lambda: W.rmat_directed(9, 8, seed=2)}[name]()
    g = W.with_weights(g, 1, 9, seed=4)
    srcs = np.random.default_rng(ns).integers(0, g.n, ns).astype(np.int32)
    ref, _ = oracle.bc(g, srcs)
    say(f"[weighted auto] {name} {ns} sources")
    with b.Graph(g) as G:
        G.run(srcs)
        got = G.scores().copy()
        assert_bc_close(got, ref)
        G.run(srcs, sigma_limit=1)  # every source with two shortest paths runs again in FP64
        assert_bc_close(G.scores(), ref)
        check_detail(g, G.detail(srcs, dump_index=ns - 1), int(srcs[-1]))
        G.run(srcs)
        assert np.array_equal(G.scores().view(np.uint64), got.view(np.uint64))
