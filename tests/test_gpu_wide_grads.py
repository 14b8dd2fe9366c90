"""The fused backward of wide representations (128 and 256) at the edges of its
64 x 64 tiles and of its column splits: one row, one row short of a tile, a
whole one, one past it, several splits with a ragged last tile.

Against the FP64 oracle on BF16-exact inputs.  An entry of G (of H = G / d
with distances) is rounded to BF16, 2^-9 relative at most, before the product;
the terms of a gradient are of its own size or add up at random: 1e-2 in the
relative 2-norm, as everywhere on this path.
"""
import numpy as np
import pytest

from tests.gpu_helpers import rel_l2
from tests.test_gpu_infonce_hooks import FUSED, _bf16_exact, _oracle, _run

pytestmark = pytest.mark.gpu

CASES = [(1, 128, "dot", "symmetric_infonce"), (17, 256, "l2", "symmetric_infonce"),
         (63, 128, "l2", "fwd_infonce"), (64, 256, "dot", "bwd_infonce"),
         (65, 128, "l2sq", "symmetric_infonce"), (65, 256, "l2", "symmetric_infonce"),
         (113, 256, "l2sq", "flatnce_bwd"), (257, 128, "l2", "symmetric_infonce"),
         (520, 256, "dot", "symmetric_infonce"), (1000, 128, "dot", "symmetric_infonce"),
         (1025, 256, "l2", "fwd_infonce"), (2111, 128, "l2", "bwd_infonce")]


@pytest.mark.parametrize("B,D,energy,loss", CASES)
def test_wide_gradients(B, D, energy, loss):
    rng = np.random.default_rng(B + D)
    x = rng.standard_normal((B, D))
    y = 0.6 * x + 0.8 * rng.standard_normal((B, D))
    scale = {"dot": 0.3, "l2": 0.5, "l2sq": 0.2}[energy]
    x, y = (_bf16_exact(scale * v) for v in (x, y))
    g, o = _run(FUSED, x, y, energy, loss), _oracle(x, y, energy, loss)
    for k in ("dphi", "dpsi"):
        if np.linalg.norm(o[k]) > 1e-12:
            assert rel_l2(g[k], o[k]) <= 1e-2, (k, rel_l2(g[k], o[k]))
        else:
            assert np.max(np.abs(g[k])) <= 1e-6
