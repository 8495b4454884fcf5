"""Loss and gradient of the policy network at the edges of its sample tiles
(64) and of its workgroups (256 tiles), against the float64 reference (rel
1e-4, abs 1e-6 as for the network's other tests), with unmeasured targets that
are not finite."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import mlp_ref
from paper_2008_05718_amd import binding as b

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 129, 4097, 16384, 16385, 16449, 40000])
def test_tiles(n):
    rng = np.random.default_rng(n)
    X = rng.uniform(0, 1, (n, b.BC_MLP_IN)).astype(np.float32)
    Y = rng.uniform(2, 10, (n, b.BC_MLP_OUT)).astype(np.float32)
    M = (rng.uniform(0, 1, (n, b.BC_MLP_OUT)) < 0.4).astype(np.uint8)
    M[0, 3] = 1
    w = mlp_ref.init(n % 7)
    L, G = mlp_ref.loss_grad(w.astype(np.float64), X.astype(np.float64), Y.astype(np.float64), M)
    Y[M == 0] = np.nan
    print(f"[mlp tiles] n={n}", flush=True)
    loss, g = b.bc_mlp_loss_grad(w, X, Y, M)
    assert abs(loss - L) <= 1e-4 * abs(L) + 1e-6
    np.testing.assert_allclose(g, G, rtol=1e-4, atol=1e-6)
    again = b.bc_mlp_loss_grad(w, X, Y, M)
    assert again[0] == loss and np.array_equal(again[1], g)
