"""The policy head where its kernel's paths change: outputs of exactly 64
columns and one action more (a column a lane up to 64, a loop above), one
action, states wider than the 512 columns requested ahead, batches that end
inside a workgroup, and split and unsplit output layers.  Bars and oracle are
those of the policy step's parity test.
"""
import pytest

from tests import test_gpu_actor as A

pytestmark = pytest.mark.gpu

CASES = [
    A.SMALL.with_(name="actor_a32", act_dim=32, batch_size=130),
    A.SMALL.with_(name="actor_a33", act_dim=33, batch_size=131),
    A.SMALL.with_(name="actor_a1", act_dim=1, batch_size=67),
    A.SMALL.with_(name="actor_s516", obs_dim=516, batch_size=65),
    A.SMALL.with_(name="actor_s507", obs_dim=507, batch_size=66, actor_hidden=(256, 256)),
    A.SMALL.with_(name="actor_a32_bf16", precision="bf16", logits="fused", act_dim=32, batch_size=259,
                  hidden=(128, 128), actor_hidden=(256, 256)),
]


@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_policy_head_at_its_edges(w, monkeypatch):
    monkeypatch.setitem(A.CASES, w.name, w)
    A.test_actor_step_matches_oracle(w.name)
