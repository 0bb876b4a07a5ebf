"""The wide resident schedule (batches past eight environments per compute unit) against the
streamed one: the same arithmetic in another arrangement, so every output is equal bit for bit."""
import pytest

from _helpers import cuda
from workload import ActorConfig, EnvConfig, make_actor_weights, make_market, pack_actor_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,D,T,I,sigma", [(2049, 30, 66, 5, 0.1), (4096, 31, 3, 5, 0.0), (4099, 28, 65, 5, 0.2),
                                           (8192, 30, 2, 5, 0.1), (8205, 29, 5, 5, 0.1), (20001, 30, 1, 5, 0.1),
                                           (2500, 25, 4, 6, 0.1)])
def test_wide_equals_streamed(N, D, T, I, sigma):
    import torch
    from paper_2501_10709_amd.vecenv import Ensemble, VecEnv
    dev = cuda()
    cfg = EnvConfig(n_envs=N, n_stocks=D, n_ind=I, n_days=T)
    m = make_market(31, D, T) if I == 5 else None
    if m is None:
        import numpy as np
        m5 = make_market(31, D, T)
        ind = np.concatenate([m5.ind, m5.ind[:, :1] * 0.5], axis=1)
        close = m5.close
    else:
        close, ind = m.close, m.ind
    w = pack_actor_weights(make_actor_weights(ActorConfig(in_dim=cfg.state_dim, hidden=256, out_dim=D, bias_std=0.1)))
    ens = Ensemble(w, 3, cfg.state_dim, 256, D, dtype="bf16", max_batch=N, device=dev)
    got = {}
    for schedule in (0, 1):
        env = VecEnv(cfg, close, ind, device=dev)
        env.set_fused_tuning(schedule=schedule)
        env.reset(return_obs=False)
        out = env.rollout(T, ens=ens, sigma=sigma, noise_key=11, env_offset=5, path="fused")
        got[schedule] = {**out, **{k: v for k, v in env.read_state().items() if k != "day"}}
    for k in got[0]:
        assert torch.equal(got[0][k], got[1][k]), (k, (got[0][k] != got[1][k]).sum().item())
    assert (got[0]["qty"] > 0).any()
