"""The generic fused schedule at the sizes where its paths part: stocks up to and past a pair of
16-lane rows, output tiles that do and do not leave wavefronts over (the sliced last layer), hidden
tiles below and past one per wavefront, actors in one and several passes, ragged tiles, and the
batched form's 32-row tiles -- against the oracle."""
import numpy as np
import pytest

from _helpers import TOL_BF16, actors_case, check_actions, check_replay, cuda, env_case

pytestmark = pytest.mark.gpu

# D, N, H, K, T
SHAPES = [(1, 1, 32, 1, 6), (16, 17, 96, 2, 8), (17, 33, 128, 3, 12), (32, 31, 224, 4, 6), (33, 16, 64, 3, 8),
          (48, 19, 288, 3, 5), (60, 15, 256, 5, 5), (128, 9, 32, 3, 3),
          # three environments a workgroup and sixteen, ragged at the end
          (20, 700, 64, 2, 5), (36, 4099, 32, 1, 3)]


def _np(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("D,N,H,K,T", SHAPES)
@pytest.mark.parametrize("batched", [False, True])
def test_generic_schedule_matches_oracle(D, N, H, K, T, batched):
    from paper_2501_10709_amd.vecenv import Batch, Ensemble, VecEnv
    if batched and H > 256:
        pytest.skip("the batch takes up to 256 hidden units")
    dev = cuda()
    S = 7 * D + 1
    cfg, m = env_case(N, D, 5, T, 77)
    acfg, actors, packed = actors_case(K, S, H, D)
    ens = Ensemble(packed, K, S, H, D, dtype="bf16", max_batch=N, device=dev)
    env = VecEnv(cfg, m.close, m.ind, device=dev)
    obs0 = _np(env.reset())
    if batched:
        batch = Batch([dict(env=env, ens=ens, n_steps=T, sigma=0.1, noise_key=7, store=("obs", "act", "rew", "qty"))])
        batch.set_tiling(32, 256)
        traj = batch.run()[0]
    else:
        traj = env.rollout(T, ens=ens, sigma=0.1, noise_key=7, path="fused")
    traj = {k: _np(v) for k, v in traj.items()}
    check_replay(cfg, m, traj, obs0)
    check_actions(actors, "bf16", traj, obs0, 0.1, 7, TOL_BF16)
    assert D == 1 or np.abs(traj["qty"]).sum() > 0
    if batched:
        batch.close()


# Around the rule for environments per workgroup: weights of up to and past 24 KB a stock at three
# environments for every compute unit, two for every one, and past twelve.
@pytest.mark.parametrize("D,N,H,K", [(8, 600, 128, 2), (8, 600, 256, 2), (8, 500, 256, 2), (8, 3100, 64, 1)])
def test_generic_schedule_environments_per_workgroup(D, N, H, K):
    from paper_2501_10709_amd.vecenv import Ensemble, VecEnv
    dev = cuda()
    S, T = 7 * D + 1, 4
    cfg, m = env_case(N, D, 5, T, 78)
    acfg, actors, packed = actors_case(K, S, H, D)
    ens = Ensemble(packed, K, S, H, D, dtype="bf16", max_batch=N, device=dev)
    env = VecEnv(cfg, m.close, m.ind, device=dev)
    obs0 = _np(env.reset())
    traj = {k: _np(v) for k, v in env.rollout(T, ens=ens, sigma=0.1, noise_key=7, path="fused").items()}
    check_replay(cfg, m, traj, obs0)
    check_actions(actors, "bf16", traj, obs0, 0.1, 7, TOL_BF16)
    assert np.abs(traj["qty"]).sum() > 0
