"""The fused backward of 64-wide representations on both sides of the batch size
up to which its blocks come from two passes (2816 where the device has 256
CUs), at block and tile edges, and beyond the one-pass kernel's 4096; and the
two passes of 32-wide ones in their one launch.

Against the FP64 oracle on BF16-exact inputs, with the bound of the other
fused gradients: an entry of G (of H = G / d with distances) is rounded to
BF16, 2^-9 relative at most, before the product, and the terms of a gradient
are of its own size or add up at random: 1e-2 in the relative 2-norm.
"""
import numpy as np
import pytest

from tests.gpu_helpers import rel_l2
from tests.test_gpu_infonce_hooks import FUSED, _bf16_exact, _oracle, _run

pytestmark = pytest.mark.gpu

CASES = [(1, 64, "l2", "symmetric_infonce"), (65, 64, "l2sq", "symmetric_infonce"),
         (256, 64, "dot", "symmetric_infonce"), (257, 64, "l2", "symmetric_infonce"),
         (300, 64, "cos", "bwd_infonce"), (1000, 64, "l2", "fwd_infonce"),
         (1023, 64, "dot", "flatnce_fwd"), (2816, 64, "l2", "symmetric_infonce"),
         (2817, 64, "dot", "symmetric_infonce"), (2900, 64, "l2sq", "symmetric_infonce"),
         (4160, 64, "l2", "symmetric_infonce"), (1, 32, "dot", "symmetric_infonce"),
         (65, 32, "l2", "symmetric_infonce"), (1100, 32, "l2sq", "bwd_infonce")]


@pytest.mark.parametrize("B,D,energy,loss", CASES)
def test_block_gradients(B, D, energy, loss):
    rng = np.random.default_rng(B + D)
    x = rng.standard_normal((B, D))
    y = 0.6 * x + 0.8 * rng.standard_normal((B, D))
    scale = {"dot": 0.3, "cos": 1.0, "l2": 0.5, "l2sq": 0.2}[energy]
    x, y = (_bf16_exact(scale * v) for v in (x, y))
    g, o = _run(FUSED, x, y, energy, loss), _oracle(x, y, energy, loss)
    for k in ("dphi", "dpsi"):
        if np.linalg.norm(o[k]) > 1e-12:
            assert rel_l2(g[k], o[k]) <= 1e-2, (k, rel_l2(g[k], o[k]))
        else:
            assert np.max(np.abs(g[k])) <= 1e-6
