"""Pull steps over runs of eight vertices from eight places: graphs whose hubs
are numbered together, with vertex counts around a wavefront's 64 and a
multiple of it, alone and in a union, against the oracle (1e-10) and, bit for
bit, against pushing."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import assert_bc_close, check_detail, say
from paper_2008_05718_amd import binding as b
from paper_2008_05718_amd import workloads as W

pytestmark = pytest.mark.gpu


def _hubs(n, seed):
    """n vertices, an eighth of them joined to about half of the others."""
    rng = np.random.default_rng(seed)
    h = max(n // 8, 1)
    u, v = [], []
    for i in range(h):
        far = rng.choice(n, size=max(n // 2, 1), replace=False)
        u.append(np.full(far.size, i))
        v.append(far)
    perm = rng.permutation(n)
    return W.csr_from_edges(n, perm[np.concatenate(u)], perm[np.concatenate(v)])


@pytest.mark.parametrize("n", [65, 127, 128, 129, 511, 512, 513, 1000])
def test_runs(n):
    g = _hubs(n, seed=n)
    u = W.union([_hubs(n, seed=1), W.grid(9), _hubs(n + 3, seed=2), _hubs(77, seed=3)])
    for what, gr in (("alone", g), ("union", u)):
        say(f"[pull runs] {what} n={gr.n}")
        srcs = np.random.default_rng(5).choice(gr.n, size=min(gr.n, 150), replace=False).astype(np.int32)
        ref, _ = oracle.bc(gr, srcs)
        with b.Graph(gr) as G:
            bits = []
            for pol in (b.BC_POLICY_FORCE_PULL, b.BC_POLICY_FORCE_PUSH_TPV):
                G.run(srcs, batch=64, policy=pol, flags=b.BC_RUN_NO_BLOCKS)
                assert_bc_close(G.scores(), ref)
                bits.append(G.scores().view(np.uint64).copy())
            assert np.array_equal(bits[0], bits[1])
            check_detail(gr, G.detail(srcs, dump_index=1, batch=64, policy=b.BC_POLICY_FORCE_PULL), int(srcs[1]))
