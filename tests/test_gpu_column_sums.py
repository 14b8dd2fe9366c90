"""The column sums that FP32 launches take beside their products: the output
layers' bias gradients, and the sums of H = (dL/dF) / d that the distance
energies subtract, against the same matrices summed in 64 bits.

Bound: the RMS error of an FP32 sum taken as 64 strided chains and a tree,
formed here on the same columns; 1.25 of it where partial sums of the split
product are rounded and added as a tree themselves.
"""
import numpy as np
import pytest
import torch

from synthetic import workloads as WL
from tests.gpu_helpers import gpu_step, setup
from tests.test_gpu_infonce_hooks import MAT, _ctx

pytestmark = pytest.mark.gpu


def _tree(m):
    """Sums over the rows of m: row i in chain i % 64, one rounding an addition."""
    f = lambda v: v.astype(np.float32).astype(np.float64)
    s = np.zeros((64, m.shape[1]))
    for i in range(0, len(m), 64):
        v = m[i:i + 64]
        s[:len(v)] = f(s[:len(v)] + v)
    while len(s) > 1:
        h = len(s) // 2
        s = f(s[:h] + s[h:])
    return s[0]


def _rms(got, m):
    return np.sqrt(np.mean((got - m.sum(0)) ** 2))


@pytest.mark.parametrize("B,D", [(250, 64), (600, 40), (1500, 64), (2600, 128)])
def test_distance_column_sums(B, D):
    # phi = 0: dpsi_jk = -(sum_i H_ij) psi_jk, so with psi_j0 = 1 the sum itself
    psi = (0.2 * np.random.default_rng(B + D).standard_normal((B, D))).astype(np.float32)
    psi[:, 0] = 1.0
    w, crit = _ctx(MAT, B, D, "l2sq", "symmetric_infonce")
    print(f"B={B} D={D}", flush=True)
    dev = torch.device("cuda:0")
    q = torch.from_numpy(psi).to(dev)
    p = torch.zeros_like(q)
    ws, lo = crit.workspace(dev), torch.zeros(8, device=dev)
    dphi, dpsi = torch.empty_like(p), torch.empty_like(q)
    crit.crl_infonce_fwd(p, q, ws, lo)
    crit.crl_infonce_bwd(p, q, ws, dphi, dpsi)
    H = crit.view(ws, "logits").double().cpu().numpy()  # the backward leaves H there
    got = -dpsi[:, 0].double().cpu().numpy()
    crit.close()
    print(f"rms {_rms(got, H):.3g}, tree {_rms(_tree(H), H):.3g}", flush=True)
    assert _rms(got, H) <= _rms(_tree(H), H)


@pytest.mark.parametrize("B,hidden", [(250, (64, 64)), (1001, (256, 256)), (4100, (512, 512))])
def test_output_bias_gradients(B, hidden):
    w = WL.SMALL_RELU.with_(name=f"bias_{B}", batch_size=B, hidden=hidden, num_envs=16, episode_len=40)
    g = gpu_step(w, *setup(w), step=3)
    for got, dz in ((g.g_phi[-1]["b"], g.dphi), (g.g_psi[-1]["b"], g.dpsi)):
        dz = dz.astype(np.float64)
        print(f"rms {_rms(got, dz):.3g}, tree {_rms(_tree(dz), dz):.3g}", flush=True)
        assert _rms(got, dz) <= 1.25 * _rms(_tree(dz), dz)
