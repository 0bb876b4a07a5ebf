"""Fused rollouts as spans of days: with the actions stored a launch runs as many days as the market
table has room for (341 at three actors of 256 units) and the noise passes through the action rows;
without them it runs 64 days on scratch.  Both give the same rewards and state, bit for bit, on each
schedule, past the end of a span and with and without noise."""
import pytest

from _helpers import actors_case, cuda, env_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,schedule", [(21, 0), (40, 1), (2100, 0)])  # resident, streamed, wide
@pytest.mark.parametrize("sigma", [0.1, 0.0])
def test_span_length_does_not_matter(N, schedule, sigma):
    import torch
    from paper_2501_10709_amd.vecenv import Ensemble, VecEnv
    dev = cuda()
    T = 350 if N < 100 else 345
    cfg, m = env_case(N, 30, 5, T, 5)
    acfg, actors, packed = actors_case(3, 211, 256, 30)
    ens = Ensemble(packed, 3, 211, 256, 30, dtype="bf16", max_batch=N, device=dev)
    got = []
    for store in (("act", "rew"), ("rew",)):
        env = VecEnv(cfg, m.close, m.ind, device=dev)
        env.set_fused_tuning(schedule=schedule)
        env.reset(return_obs=False)
        out = env.rollout(T, ens=ens, sigma=sigma, noise_key=3, path="fused", store=store)
        got.append({"rew": out["rew"], **{k: v for k, v in env.read_state().items() if k != "day"}})
    for k in got[0]:
        assert torch.equal(got[0][k], got[1][k]), k
    assert (got[0]["rew"] != 0).any()
