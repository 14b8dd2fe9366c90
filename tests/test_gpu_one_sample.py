"""One sample without the penalty: the softmax of one logit is 1, so the InfoNCE
gradients of the materialised matrix vanish, whatever the energy."""
import numpy as np
import pytest

from tests.test_gpu_infonce_hooks import MAT, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("energy", ["dot", "l2", "l2sq", "cos", "l1"])
@pytest.mark.parametrize("loss", ["fwd_infonce", "symmetric_infonce", "bwd_infonce"])
@pytest.mark.parametrize("D", [8, 72])
def test_gradients_of_one_sample_vanish(energy, loss, D):
    rng = np.random.default_rng(D)
    x, y = (rng.standard_normal((1, D)).astype(np.float32) for _ in range(2))
    g = _run(MAT, x, y, energy, loss, beta=0.0)
    # r = c = F_ii: exp of 0 is 1 and its logarithm 0
    assert abs(g["loss"][0]) <= 1e-6
    for k in ("dphi", "dpsi"):
        assert np.max(np.abs(g[k])) <= 1e-6, k
