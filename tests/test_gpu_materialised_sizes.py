"""The materialised FP32 critic matrix at the sizes where its launches change:
one row, chunk and tile edges, the column merge inside the loss kernel (up to
B = 2048) and apart from it, split and unsplit dphi / dpsi products, and the
L1 backward with one and several splits of its sums.

Against the FP64 oracle.  FP32 sums of at most 2600 terms in short chains err
by some 1e-6 relative, a distance from the norm expansion by some 1e-5 of the
entries near its floor: 1e-4 on the loss parts, r, c and both gradients
(relative 2-norm).
"""
import numpy as np
import pytest

from tests.gpu_helpers import rel_l2
from tests.test_gpu_infonce_hooks import MAT, _oracle, _run

pytestmark = pytest.mark.gpu

CASES = [(1, 8, "l2", "symmetric_infonce"), (2, 40, "l1", "fwd_infonce"),
         (15, 16, "cos", "symmetric_infonce"), (63, 264, "l2sq", "bwd_infonce"),
         (65, 32, "l1", "symmetric_infonce"), (257, 72, "l2", "dpo"),
         (300, 256, "l1", "ipo"), (513, 64, "dot", "symmetric_infonce"),
         (1025, 48, "l2", "symmetric_infonce"), (1100, 40, "l1", "sppo"),
         (2048, 64, "cos", "flatnce_bwd"), (2049, 64, "l2", "symmetric_infonce"),
         (2600, 24, "dot", "fb")]


@pytest.mark.parametrize("B,D,energy,loss", CASES)
def test_materialised_sizes(B, D, energy, loss):
    rng = np.random.default_rng(B + D)
    x = rng.standard_normal((B, D))
    y = 0.6 * x + 0.8 * rng.standard_normal((B, D))
    scale = {"dot": 0.5, "cos": 1.0, "l2": 1.0, "l2sq": 0.2, "l1": 0.2}[energy]
    x, y = (scale * v.astype(np.float32) for v in (x, y))
    g, o = _run(MAT, x, y, energy, loss), _oracle(x, y, energy, loss)
    for i, k in enumerate(("total", "fwd", "bwd", "pen")):
        assert abs(g["loss"][i] - o[k]) <= 1e-4 * max(abs(o[k]), 1.0), (k, g["loss"][i], o[k])
    for k in ("r", "c", "dphi", "dpsi"):
        if np.linalg.norm(o[k]) > 1e-12:
            assert rel_l2(g[k], o[k]) <= 1e-4, (k, rel_l2(g[k], o[k]))
