"""The engine that a weighted run takes when weighted_lanes is left open, by
arcs, sources and depth: a batch of up to 64 sources on the whole GPU (counted
in n_batches), a source per workgroup, or 16 per workgroup (which alone counts
relaxed pairs with n_batches at zero).  The engine is asserted, the scores are
compared with the oracle within 1e-10 relative (non-negative terms), and
distances and path counts as everywhere."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, check_detail, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


def _grid(rows, cols, extra=0):
    """A rows x cols grid and `extra` vertices without arcs."""
    ids = np.arange(rows * cols).reshape(rows, cols)
    u = np.concatenate([ids[:, :-1].ravel(), ids[:-1].ravel()])
    v = np.concatenate([ids[:, 1:].ravel(), ids[1:].ravel()])
    return W.csr_from_edges(rows * cols + extra, u, v)


def _path(n):
    return W.csr_from_edges(n, np.arange(n - 1), np.arange(1, n))


def _star_and_path():
    # the vertex of largest degree sees one hop; the depth is in another component
    n = 20000
    return W.csr_from_edges(n + 50, np.concatenate([np.arange(n - 1), np.full(49, n)]),
                            np.concatenate([np.arange(1, n), np.arange(n + 1, n + 50)]))


def _degrees():
    rng = np.random.default_rng(3)
    degrees = [1, 2, 63, 64, 65, 127, 128, 1023, 1024, 1025, 2049, 2500]
    pool = 2600
    u = np.concatenate([np.full(d, pool + i) for i, d in enumerate(degrees)] + [rng.integers(0, pool, 9000)])
    v = np.concatenate([rng.choice(pool, d, replace=False) for d in degrees] + [rng.integers(0, pool, 9000)])
    return W.csr_from_edges(pool + len(degrees), u, v)


GRAPHS = {
    "rmat12": (lambda: W.rmat(12, 16, seed=31), 30),
    "rmat14": (lambda: W.rmat(14, 16, seed=31), 30),
    "directed13": (lambda: W.rmat_directed(13, 16, seed=31), 30),
    "degrees": (_degrees, 2),
    "path600": (lambda: _path(600), 9),
    "path20000": (lambda: _path(20000), 9),
    "star+path": (_star_and_path, 9),
    "grid70": (lambda: _grid(70, 70), 30),
    "grid200": (lambda: _grid(200, 200), 30),
    "grid20x2000": (lambda: _grid(20, 2000, extra=1), 30),
}


def _engine(st):
    if st["n_batches"]:
        return "wide"
    return "sixteen" if st["phase_lane_arcs"][1] else "one"


@pytest.mark.parametrize("name,ns,engine", [
    ("rmat12", 64, "wide"), ("rmat12", 1024, "one"), ("rmat14", 256, "wide"), ("directed13", 65, "wide"),
    ("degrees", 62, "wide"), ("path600", 64, "one"), ("path600", 2560, "one"), ("path600", 2561, "sixteen"),
    ("path20000", 8, "one"), ("path20000", 64, "one"), ("star+path", 64, "one"), ("grid70", 64, "one"),
    ("grid200", 64, "wide"), ("grid200", 256, "one"), ("grid20x2000", 12, "wide"),
])
def test_engine_by_arcs_sources_and_depth(name, ns, engine):
    make, wmax = GRAPHS[name]
    g = W.with_weights(make(), 1, wmax, seed=5)
    srcs = np.random.default_rng(ns).integers(0, g.n, ns).astype(np.int32)
    if name == "grid20x2000":
        srcs[3] = g.n - 1  # the vertex without arcs
    few = srcs[:: max(1, ns // 12)]
    with b.Graph(g) as G:
        G.run(srcs)
        st = G.stats()
        say(f"[weighted choice] {name} {ns}: {_engine(st)} {st['ms']:.1f} ms")
        assert _engine(st) == engine
        got = G.scores().copy()
        assert_bc_close(got, oracle.bc_sliced(g, srcs, threads=8)[0])
        G.run(srcs)
        assert np.array_equal(G.scores().view(np.uint64), got.view(np.uint64))
        if engine == "wide":
            check_detail(g, G.detail(srcs, ns - 1), int(srcs[-1]))
    with b.Graph(g, flags=b.BC_KEEP_ORDER) as G:  # the depth is known there, too
        G.run(srcs)
        assert _engine(G.stats()) == engine
        G.run(few, weighted_lanes=1)
        assert_bc_close(G.scores(), oracle.bc_sliced(g, few, threads=8)[0])


def test_wide_engine_beyond_64_bits():
    # path counts of a 200 x 200 grid of unit weights leave 64 bits from every
    # corner and not from the middle
    g = W.with_weights(_grid(200, 200), 1, 1, seed=2)
    srcs = np.array([0, 199, 100 * 200 + 100, 200 * 200 - 1, 0], np.int32)
    ref, modes = oracle.bc(g, srcs)
    assert modes[0] == 1
    with b.Graph(g) as G:
        G.run(srcs)
        st = G.stats()
        assert _engine(st) == "wide" and st["f64_sources"] == int(modes.sum())
        assert_bc_close(G.scores(), ref)
        check_detail(g, G.detail(srcs, 0), 0)
        G.run(srcs, flags=b.BC_RUN_FORCE_F64)
        assert _engine(G.stats()) == "wide"
        assert_bc_close(G.scores(), ref)
