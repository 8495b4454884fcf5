"""Handles share the streams their concurrent parts run on: handles used in
turn, from several threads at once and across the destruction of another one
give the bits that a handle alone gives (a handle's scores do not depend on
which stream its parts ran on)."""
from __future__ import annotations

import threading

import numpy as np
import pytest

from gpu_util import say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(G, srcs):
    G.run(srcs, batch=64, flags=b.BC_RUN_NO_BLOCKS)
    return G.scores().view(np.uint64).copy()


@pytest.mark.parametrize("rounds", [1, 4])
def test_handles_in_turn_and_at_once(rounds):
    graphs = [W.rmat(10, 8, seed=1), W.union([W.barabasi_albert(300 + 40 * i, 3, seed=i) for i in range(12)]),
              W.grid(40, 0.05, 0.01, seed=2)]
    srcs = [W.choose_sources(g, min(g.n - 50, 700), seed=4) for g in graphs]
    want = []
    for g, s in zip(graphs, srcs):  # one handle alive at a time
        with b.Graph(g) as G:
            want.append(_run(G, s))
    handles = [b.Graph(g) for g in graphs]
    try:
        for r in range(rounds):
            say(f"[part streams] round {r}: in turn, then at once")
            for G, s, w in zip(handles, srcs, want):
                assert np.array_equal(_run(G, s), w)
            got = [None] * len(handles)

            def work(i):
                got[i] = _run(handles[i], srcs[i])

            th = [threading.Thread(target=work, args=(i,)) for i in range(len(handles))]
            for t in th:
                t.start()
            for t in th:
                t.join()
            for x, w in zip(got, want):
                assert np.array_equal(x, w)
        handles.pop(0).close()  # the others go on
        for G, s, w in zip(handles, srcs[1:], want[1:]):
            assert np.array_equal(_run(G, s), w)
    finally:
        for G in handles:
            G.close()
    with b.Graph(graphs[0]) as G:  # and a first one again after the last
        assert np.array_equal(_run(G, srcs[0]), want[0])
