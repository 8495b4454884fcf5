"""Loss and gradient of the policy network near the ends of the FP32 range,
where a sum over the samples leaves it and the mean does not, against the
float64 reference (rel 1e-4 as for the network's other tests)."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import mlp_ref
from paper_2008_05718_amd import binding as b

pytestmark = pytest.mark.gpu


# targets around 3e17: squares of 1e35, 64 samples of them beyond 3.4e38; around
# 1e34: gradients in range, the loss (5e67) is not
@pytest.mark.parametrize("size", [1.0, 3e17, 1e34])
@pytest.mark.parametrize("n,share", [(1, 1.0), (65, 1.0), (16384, 1.0), (16384, 0.001), (40000, 0.4)])
def test_means_whose_sums_leave_the_range(n, share, size):
    rng = np.random.default_rng(n)
    X = rng.uniform(0, 1, (n, b.BC_MLP_IN)).astype(np.float32)
    Y = (rng.uniform(1, 2, (n, b.BC_MLP_OUT)) * size).astype(np.float32)
    M = (rng.uniform(0, 1, (n, b.BC_MLP_OUT)) < share).astype(np.uint8)
    M[0, 3] = 1
    w = mlp_ref.init(n % 7)
    L, G = mlp_ref.loss_grad(w.astype(np.float64), X.astype(np.float64), Y.astype(np.float64), M)
    print(f"[mlp range] n={n} share={share} size={size}: loss {L:.3e}, gradient up to {np.abs(G).max():.3e}", flush=True)
    loss, g = b.bc_mlp_loss_grad(w, X, Y, M)
    if L < 3e38:
        assert abs(loss - L) <= 1e-4 * L
    else:
        assert np.isinf(loss)
    np.testing.assert_allclose(g, G, rtol=1e-4, atol=1e-4 * np.abs(G).max() * 2.0 ** -10)
