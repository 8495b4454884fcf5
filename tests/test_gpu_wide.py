"""Weighted graphs with the engine left to choose (a batch of up to 64 sources
on the whole GPU): list lengths around its row widths (8, 16, 32, 64), degree
classes around its packing (64 arcs) and segments (1024 arcs), both
directions, path counts beyond the limit and beyond 64 bits, long paths, and a
memory cap under which it does not fit.  Distances and uint64 counts bit for
bit, FP64 values within 1e-10 relative (sums of non-negative terms: error about
(rounds + degree) * 2^-53); runs repeat bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, check_detail, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


def _check(g, srcs, dumps, **opts):
    ref, modes = oracle.bc(g, srcs)
    with b.Graph(g) as G:
        G.run(srcs, **opts)
        got = G.scores().copy()
        st = G.stats()
        assert_bc_close(got, ref)
        G.run(srcs, flags=b.BC_RUN_NO_GRAPHS, **opts)
        assert np.array_equal(G.scores(), got)
        for i in dumps:
            check_detail(g, G.detail(srcs, i, **opts), int(srcs[i]))
            assert np.array_equal(G.scores(), got)
    return st, modes


@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("k", [1, 8, 9, 16, 17, 32, 33, 64, 65, 200])
def test_list_lengths(k, directed):
    base = W.rmat_directed(13, 16, seed=31) if directed else W.rmat(12, 16, seed=31)
    g = W.with_weights(base, 1, 30, seed=5)
    srcs = W.choose_sources(base, 200, seed=6)[:k]
    say(f"[wide] k={k} directed={directed}")
    st, _ = _check(g, srcs, {0, k - 1})
    # n_batches counts this engine's batches only (about 100,000 arcs carry two of 64)
    if k <= 128:
        assert st["n_batches"] == -(-k // (8 if k <= 8 else 16 if k <= 16 else 32 if k <= 32 else 64))


@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("wmax", [1, 2, 1 << 30])
def test_degree_classes_and_weights(wmax, directed):
    rng = np.random.default_rng(3)
    degrees = [1, 2, 63, 64, 65, 127, 128, 1023, 1024, 1025, 2049, 2500]
    pool = 2600
    n = pool + len(degrees)
    u = [np.full(d, pool + i) for i, d in enumerate(degrees)] + [rng.integers(0, pool, 9000)]
    v = [rng.choice(pool, d, replace=False) for d in degrees] + [rng.integers(0, pool, 9000)]
    u, v = np.concatenate(u), np.concatenate(v)
    if directed:
        flip = rng.random(u.size) < 0.5
        base = W.digraph_from_arcs(n, np.where(flip, v, u), np.where(flip, u, v))
    else:
        base = W.csr_from_edges(n, u, v)
    g = W.with_weights(base, 1, wmax, seed=8)
    srcs = np.concatenate([np.arange(pool, n), rng.choice(pool, 50, replace=False)]).astype(np.int32)
    say(f"[wide] degree classes wmax={wmax} directed={directed}")
    _check(g, srcs, (0, 9, 11, 40))


def test_overflow_limit_and_fp64():
    base = W.grid(70)
    g = W.with_weights(base, 1, 1, seed=2)
    srcs = np.array([0, 69, 35 * 70 + 35, 70 * 70 - 1, 100, 0], np.int32)
    st, modes = _check(g, srcs, (0, 2))
    assert modes[0] == 1 and st["f64_sources"] == int(modes.sum())
    base = W.rmat(11, 16, seed=64)
    g = W.with_weights(base, 1, 2, seed=8)
    srcs = W.choose_sources(base, 60, seed=9)
    lim = 195
    over = sum(bool((oracle.source(g, int(s)).sigma_u64 > lim).any()) for s in srcs)
    assert 0 < over < len(srcs)
    ref, _ = oracle.bc(g, srcs)
    with b.Graph(g) as G:
        G.run(srcs, sigma_limit=lim)
        assert G.stats()["f64_sources"] == over
        assert_bc_close(G.scores(), ref)
        G.run(srcs, flags=b.BC_RUN_FORCE_F64)
        assert_bc_close(G.scores(), ref)


def test_long_path_accumulate_and_isolated():
    n = 14000
    u = np.arange(n - 2)
    base = W.csr_from_edges(n, u, u + 1)  # the last vertex is isolated
    g = W.with_weights(base, 1, 9, seed=5)
    srcs = np.array([0, n - 1, 700, 700, n - 2], np.int32)
    ref, _ = oracle.bc(g, srcs)
    with b.Graph(g) as G:
        G.run(srcs[:3])
        G.run(srcs[3:], flags=b.BC_RUN_ACCUMULATE)
        assert_bc_close(G.scores(), ref)
        G.run([n - 1])
        assert not G.scores().any()


def test_memory_cap_falls_back():
    base = W.rmat(11, 16, seed=65)
    g = W.with_weights(base, 1, 50, seed=9)
    srcs = W.choose_sources(base, 60, seed=10)
    ref, _ = oracle.bc(g, srcs)
    with b.Graph(g) as G:
        floor = G.info()["device_bytes"]
        ran = 0
        for mib in range(1, 16):
            G.set_device_limit(floor + (mib << 20))
            try:
                G.run(srcs)
            except b.BCError as e:
                assert e.status == 3
            else:
                ran += 1
                assert_bc_close(G.scores(), ref)
            assert G.info()["device_bytes"] <= floor + (mib << 20)
        assert ran
