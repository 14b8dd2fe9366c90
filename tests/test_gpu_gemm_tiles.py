"""GPU parity of the encoder and logit GEMMs at the edges of their tiles.

The GEMM takes tiles of edge 32, 64 or 128 by the size of the launch; batch,
widths and depths here sit one below, on and one above those edges, with K
ranges that are no whole stages (64 BF16 or 32 FP32 values), against the FP64
oracle.  Tolerances: FP32 sums of K <= 4200 products in chains of 128 (relative
error some 1e-6) get 1e-4 on the loss and cosine 0.99999 on every gradient;
BF16 operands (8-bit mantissas, 1e-2 on the activations) 1e-2 and 0.999.
"""
import pytest
import torch

from synthetic import critic_params_for
from synthetic import workloads as WL
from tests.gpu_helpers import compare, gpu_step, oracle_step, print_report, setup

pytestmark = pytest.mark.gpu

_F = WL.SMALL_RELU.with_(num_envs=16, episode_len=40, energy_function="dot")
_L = WL.LN_FWD_FP32.with_(num_envs=16, episode_len=40)
_H = WL.DOT_B4096_BF16.with_(num_envs=16, episode_len=40)
CASES = [
    # FP32, edge 32: one row, one below / on / above an edge, a single K chunk
    _F.with_(batch_size=1, hidden=(8,), repr_dim=8),
    _F.with_(batch_size=31, hidden=(40, 40), repr_dim=24),
    _L.with_(batch_size=32, hidden=(32, 32), repr_dim=32),
    _F.with_(batch_size=33, hidden=(72,), repr_dim=8, energy_function="l2"),
    _L.with_(batch_size=129, hidden=(136, 136), repr_dim=40, energy_function="cos"),
    _F.with_(batch_size=257, hidden=(264, 264), energy_function="l2sq",
             contrastive_loss_function="dpo"),
    # FP32, edge 64 (ragged rows and columns, K of 1000 and 1001)
    _L.with_(batch_size=1001, hidden=(1000, 1000)),
    # FP32, edge 128
    _F.with_(batch_size=4200, hidden=(1016,), repr_dim=72),
    # BF16, edges 32 and 64, with a K of 40, 200 and a batch that is no whole stage
    _H.with_(batch_size=1, hidden=(64,), repr_dim=32),
    _H.with_(batch_size=63, hidden=(40, 40), repr_dim=32),
    _H.with_(batch_size=190, hidden=(200, 200), repr_dim=128, energy_function="l2"),
    _H.with_(batch_size=1001, hidden=(512, 512), repr_dim=32),
    # BF16, edge 128 with a ragged batch
    _H.with_(batch_size=2113, hidden=(1024, 1024)),
]
CASES = [w.with_(name=f"b{w.batch_size}_{w.activation}_h{len(w.hidden)}x{w.hidden[0]}_d{w.repr_dim}"
                      f"_{w.energy_function}_{w.precision}") for w in CASES]


@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_critic_parity_at_tile_edges(w):
    obs, act, phi, psi = setup(w)
    g = gpu_step(w, obs, act, phi, psi, step=3)
    o = oracle_step(w, obs, act, phi, psi, step=3)
    rep = compare(w, g, o)
    print_report(w.name, rep)
    loss, cos = (1e-4, 0.99999) if w.precision == "fp32" else (1e-2, 0.999)
    for i, k in enumerate(("total", "fwd", "bwd", "pen")):
        assert abs(g.loss[i] - o[k]) <= loss * max(abs(o[k]), 1.0), (k, g.loss[i], o[k])
    if w.batch_size > 1:  # one sample: gradients of the InfoNCE part are zero
        assert rep["min_cos"] >= cos


def test_input_padding_is_not_read_in_fp32():
    """Columns of x_sa and x_g past the real width never reach a result."""
    from paper_2408_11052_amd import Critic
    w = _L.with_(name="padding", batch_size=70, hidden=(64, 64))
    dev = torch.device("cuda:0")
    crit = Critic(w)
    params = torch.from_numpy(crit.pack(*critic_params_for(w, seed=1, perturb=0.1))).to(dev)
    ws = crit.workspace(dev)
    out = []
    for pad in (0.0, float("nan")):
        x_sa, x_g, _ = crit.inputs(dev)
        gen = torch.Generator(device=dev).manual_seed(5)
        for x, n in ((x_sa, w.in_sa), (x_g, w.goal_dim)):
            x.fill_(pad)
            x[:, :n] = torch.randn(w.batch_size, n, generator=gen, device=dev)
        loss = torch.zeros(8, device=dev)
        grads = torch.empty(crit.nparam, device=dev)
        crit.crl_critic_fwd(params, None, x_sa, x_g, ws, loss)
        crit.crl_critic_bwd(params, None, x_sa, x_g, ws, grads)
        torch.cuda.synchronize()
        out.append((loss, grads))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    crit.close()
