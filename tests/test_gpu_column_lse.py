"""Column log-sum-exps of the materialised critic matrix, against those of the
same FP32 matrix taken in 64 bits.  Rows and columns hold the same number of
exponentials and end in the same logarithm, so for a matrix with like rows and
columns the columns' error is the rows'; 1.05 covers the sample of a thousand
or more of each.  Up to B = 256 the loss kernel merges the columns' chunks, above a
kernel of its own.
"""
import numpy as np
import pytest
import torch

from tests.test_gpu_infonce_hooks import MAT, _ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,D,energy,scale", [(256, 64, "l2sq", 0.3), (257, 64, "l2sq", 0.3),
                                              (1024, 64, "l2sq", 0.3), (2048, 64, "l2sq", 0.3),
                                              (2048, 64, "dot", 0.5), (2049, 64, "dot", 0.5)])
def test_columns_err_like_rows(B, D, energy, scale):
    w, crit = _ctx(MAT, B, D, energy, "symmetric_infonce")
    dev = torch.device("cuda:0")
    ws, lo = crit.workspace(dev), torch.zeros(8, device=dev)
    err = {"row_lse": [], "col_lse": []}
    for seed in range(6):
        gen = torch.Generator(device=dev).manual_seed(seed)
        p, q = (scale * torch.randn(B, D, generator=gen, device=dev) for _ in range(2))
        crit.crl_infonce_fwd(p, q, ws, lo)
        F = crit.view(ws, "logits").double()
        for dim, k in ((1, "row_lse"), (0, "col_lse")):
            err[k].append((crit.view(ws, k).double() - torch.logsumexp(F, dim)).cpu().numpy())
    crit.close()
    rms = {k: float(np.sqrt(np.mean(np.square(v)))) for k, v in err.items()}
    print(B, D, energy, rms, flush=True)
    assert rms["col_lse"] <= 1.05 * rms["row_lse"]
