"""The autotuner on graphs whose runs choose the width of a batch themselves:
the result leaves it open, and a tuned run of another list has the batches
that an untuned one has.  Scores against the oracle within 1e-10 relative."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns", [2048, 4096, 8192])
def test_tuned_runs_choose_their_width_by_the_list(ns):
    g = W.erdos_renyi(1200, 6.0, seed=5)
    rng = np.random.default_rng(ns)
    srcs = rng.integers(0, g.n, ns).astype(np.int32)
    ref, _ = oracle.bc(g, srcs)
    with b.Graph(g) as G:
        G.run(srcs)
        batches = G.stats()["n_batches"]
        best = G.autotune(srcs[:2048])  # 8 lanes are the fastest for these
        say(f"[autotune open] {ns}: {best}")
        G.run(srcs, flags=b.BC_RUN_TUNED)
        assert G.stats()["n_batches"] == batches
        assert_bc_close(G.scores(), ref)
        again = G.autotune(srcs[:2048])  # from the cache
        assert again == best and best["batch"] == 0
        G.autotune(srcs[:2048], batch=1, flags=b.BC_TUNE_FRESH)  # the per-source engine, as asked for
        G.run(srcs[:20], flags=b.BC_RUN_TUNED)
        assert G.stats()["batch"] == 1


def test_general_engine_keeps_a_fixed_width():
    g = W.rmat(12, 16, seed=8)
    srcs = W.choose_sources(g, 256, seed=9)
    with b.Graph(g) as G:
        assert G.autotune(srcs, flags=b.BC_TUNE_FRESH)["batch"] in (1, 8, 16, 32, 64)
