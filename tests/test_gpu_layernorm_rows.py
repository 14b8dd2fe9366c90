"""GPU parity of the LayerNorm kernels where their rows and chunks end.

A lane owns chunks of 8 features, 64 lanes to a chunk row: widths of one chunk,
one below, on and one above 512 (where a second chunk row begins) and the
widest.  A workgroup of the backward takes 16 rows a round, and from B = 4097
on two rounds: batches end inside a wavefront's rows, in the first wavefront of
a workgroup and in the second round.  The oracle is FP64; tolerances: FP32 sums
over at most 1024 features and 4113 rows (relative error some 1e-6) get 1e-4 on
the loss and cosine 0.99999 on every gradient; BF16 operands (8-bit mantissas,
1e-2 on the activations) 1e-2 and 0.999.
"""
import pytest

from synthetic import workloads as WL
from tests.gpu_helpers import compare, gpu_step, oracle_step, print_report, setup

pytestmark = pytest.mark.gpu

_L = WL.LN_FWD_FP32.with_(num_envs=16, episode_len=40)
_H = WL.DOT_B4096_BF16.with_(num_envs=16, episode_len=40)
CASES = [
    (_L, 18, 8), (_L, 17, 504), (_L, 31, 512), (_L, 1026, 520), (_L, 2050, 1016), (_L, 2051, 1024),
    (_L, 4113, 72), (_L, 4113, 512),
    (_H, 18, 504), (_H, 67, 512), (_H, 4113, 512), (_H, 4098, 520), (_H, 4113, 1024),
]


@pytest.mark.parametrize("base,batch,width", CASES,
                         ids=[f"{w.precision}_b{b}_h{n}" for w, b, n in CASES])
def test_critic_parity_at_row_ends(base, batch, width):
    w = base.with_(name=f"ln_{base.precision}_b{batch}_h{width}", batch_size=batch, hidden=(width, width))
    obs, act, phi, psi = setup(w)
    g = gpu_step(w, obs, act, phi, psi, step=3)
    o = oracle_step(w, obs, act, phi, psi, step=3)
    rep = compare(w, g, o)
    print_report(w.name, rep)
    loss, cos = (1e-4, 0.99999) if w.precision == "fp32" else (1e-2, 0.999)
    for i, k in enumerate(("total", "fwd", "bwd", "pen")):
        assert abs(g.loss[i] - o[k]) <= loss * max(abs(o[k]), 1.0), (k, g.loss[i], o[k])
    assert rep["min_cos"] >= cos
