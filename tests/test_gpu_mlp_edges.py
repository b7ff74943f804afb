"""GPU tests of the cost model's kernels at the sizes where their loops change: a wavefront's two
samples, a gradient chain's 32 samples read ahead, a staged chunk of 256 and a full grid of 4,096."""
import numpy as np
import pytest

import workloads
import paper_2009_07482_amd as psc
from oracle import mlp as omlp
from gpu_helpers import normwise

pytestmark = pytest.mark.gpu

F = psc.PSC_FEATURES


@pytest.mark.parametrize("n", [1, 2, 3, 31, 32, 33, 255, 256, 257, 513, 4096, 4099])
def test_gradient_and_prediction_edges(n):
    """A gradient entry is one FP32 chain of n products of errors and activations: its rounding
    grows with the chain as a random walk, about sqrt(n) 2^-24 of the terms' size, and the sum can
    be smaller than its terms' size by up to sqrt(n) again (n 2^-24 = 2.4e-4 at n = 4096)."""
    g = np.random.default_rng(100 + n)
    x = g.normal(0.0, 1.0, size=(n, F)).astype(np.float32)
    t = (0.8 * x[:, 0] - 0.5 * x[:, 3] * x[:, 4] + 0.3 * x[:, 11] ** 2).astype(np.float32)
    p = workloads.mlp_init(21, F)
    m = psc.psc_mlp_create(0)
    try:
        psc.psc_mlp_set_params(m, psc.mlp_flatten(p))
        y0, cache = omlp.forward(p, x)
        assert normwise(psc.psc_mlp_predict(m, x), y0) < 1e-5
        got, loss = psc.psc_mlp_grad(m, x, t)
        assert loss == pytest.approx(omlp.loss(y0, t), rel=1e-5)
        ref = omlp.backward(p, cache, y0, t)
        got = psc.mlp_unflatten(got)
        for k in omlp.NAMES:
            assert normwise(got[k], ref[k].reshape(got[k].shape)) < max(1e-4, n * 2.0 ** -24), k
    finally:
        psc.psc_mlp_destroy(m)
