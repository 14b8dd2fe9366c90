"""The L1 backward passes a non-finite row on to every gradient entry that its
terms reach: an entry is -sum_y C(x, y) sign(d) with C NaN, which is NaN
whatever the sign, also where the feature's own difference d is NaN or 0.
"""
import numpy as np
import pytest

from tests.test_gpu_infonce_hooks import MAT, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("B,D", [(9, 8), (70, 40), (300, 64)])
def test_a_non_finite_feature_reaches_every_entry(B, D, value):
    rng = np.random.default_rng(B + D)
    x, y = (0.2 * rng.standard_normal((B, D)).astype(np.float32) for _ in range(2))
    x[:, 3] = y[:, 3] = 0.25  # a feature whose differences are all 0
    x[B // 2, 5] = value
    g = _run(MAT, x, y, "l1", "fwd_infonce")
    # the forward objective's G: row B // 2 is NaN, the others are finite
    assert np.isnan(g["dphi"][B // 2]).all()
    assert np.isnan(g["dpsi"]).all()
    assert np.isfinite(np.delete(g["dphi"], B // 2, 0)).all()
