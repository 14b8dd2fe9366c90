"""The samplers at the batch sizes where a wavefront's share changes (one, two
or four samples from 2048 and 8192 on), with a last wavefront that is partly
filled, and with a threshold table of one level, two and more: indices equal
to the oracle's, rows equal to the rows of those indices (FP32: copies).
"""
import numpy as np
import pytest
import torch

from oracle import relabel as orelabel
from oracle.replay import RingBuffer, ring_relabel_indices
from synthetic import make_buffer
from synthetic import workloads as WL
from synthetic.trajectories import unroll_stream

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

CASES = [(1, 2), (2047, 40), (2048, 66), (2051, 300), (8191, 300), (8193, 1000), (8194, 5000)]


def _inputs(B, T, **kw):
    from paper_2408_11052_amd import Critic
    w = WL.SMALL_RELU.with_(name="sizes", batch_size=B, num_envs=13, episode_len=T,
                            obs_dim=70, act_dim=3, goal_dim=5, **kw)
    crit = Critic(w)
    return w, crit, crit.inputs(), torch.full((B, 3), -7, dtype=torch.int32, device=DEV)


def _check(w, idx, x, want_idx, obs, act):
    assert np.array_equal(idx.cpu().numpy(), want_idx)
    e, t, g = (want_idx[:, k] for k in range(3))
    s, a = obs[e, t], act[e, t]
    goal = obs[e, g][:, w.goal_lo:w.goal_lo + w.goal_dim]
    for got, want in zip(x, (np.concatenate([s, a], 1), goal, np.concatenate([s, goal], 1))):
        got = got.float().cpu().numpy()
        assert np.array_equal(got[:, :want.shape[1]], want)
        assert not got[:, want.shape[1]:].any()


@pytest.mark.parametrize("B,T", CASES)
def test_episode_sampler(B, T):
    w, crit, x, idx = _inputs(B, T)
    obs, act = make_buffer(w.num_envs, T, w.obs_dim, w.act_dim)
    step = torch.full((1,), 9, dtype=torch.int64, device=DEV)
    crit.crl_sample_relabel(torch.from_numpy(obs).to(DEV), torch.from_numpy(act).to(DEV), 5, step,
                            idx, *x)
    torch.cuda.synchronize()
    want = orelabel.relabel_indices(w.num_envs, T, B, w.discounting, 5, 9)
    _check(w, idx, x, want, obs, act)


@pytest.mark.parametrize("B,T", CASES[1:6])
def test_ring_sampler(B, T):
    from paper_2408_11052_amd import ReplayRing
    w, crit, x, idx = _inputs(B, T)
    C = max(T // 2, 30)
    obs, act, traj = unroll_stream(w.num_envs, C + 17, w.obs_dim, w.act_dim, (2, T), seed=B)
    ring = ReplayRing(w.num_envs, C, w.obs_dim, w.act_dim)
    ref = RingBuffer(w.num_envs, C, w.obs_dim, w.act_dim)
    for sl in (slice(0, C), slice(C, C + 17)):
        ring.insert(*(torch.from_numpy(np.ascontiguousarray(v[sl])).to(DEV)
                      for v in (obs, act, traj)))
        ref.insert(obs[sl], act[sl], traj[sl])
    step = torch.full((1,), 4, dtype=torch.int64, device=DEV)
    ring.sample_relabel(crit, 11, step, idx, *x)
    torch.cuda.synchronize()
    want = ring_relabel_indices(ref, B, w.discounting, T, 11, 4)
    _check(w, idx, x, want, ref.obs, ref.act)
