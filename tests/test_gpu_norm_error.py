"""The squared norms of the materialised distance energies: with the other side
all zero the diagonal of the critic matrix is minus the row's own norm.

Bound: the RMS error of the FP32 sum that a wavefront takes over a row (64
strided chains of fused multiply-adds, then a tree), formed here on the same
rows.  The kernel rounds four squares at a time and the total, which is less.
"""
import numpy as np
import pytest

from tests.test_gpu_infonce_hooks import MAT, _run

pytestmark = pytest.mark.gpu


def _tree(x):
    x = x.astype(np.float32)
    s = np.zeros((len(x), 64))
    for d in range(0, x.shape[1], 64):
        v = x[:, d:d + 64].astype(np.float64)
        s[:, :v.shape[1]] += v * v
        s = s.astype(np.float32).astype(np.float64)  # one rounding a multiply-add
    while s.shape[1] > 1:
        h = s.shape[1] // 2
        s = (s[:, :h] + s[:, h:]).astype(np.float32).astype(np.float64)
    return s[:, 0]


@pytest.mark.parametrize("side", ["phi", "psi"])
@pytest.mark.parametrize("B,D", [(300, 64), (600, 40), (600, 256), (1500, 128), (4100, 64)])
def test_norms_err_less_than_a_tree(B, D, side):
    x = np.random.default_rng(B + D).standard_normal((B, D)).astype(np.float32)
    z = np.zeros_like(x)
    g = _run(MAT, *((x, z) if side == "phi" else (z, x)), energy="l2sq")
    exact = (x.astype(np.float64) ** 2).sum(1)
    rms = lambda n: np.sqrt(np.mean(((n - exact) / exact) ** 2))
    print(f"rms {rms(-g['diag']) * 2 ** 24:.3f}, tree {rms(_tree(x)) * 2 ** 24:.3f} (2^-24)", flush=True)
    assert rms(-g["diag"]) <= rms(_tree(x))
