"""The learner on the GPU (include/learner.h) against the oracle: the policy gradient of eq. (4)
with the KL diversity term of eq. (5), computed from a real rollout's stored states and rewards.

Tolerance: float32 forward and backward passes (fixed summation orders) against float64; every
entry within 1e-5 of the largest entry of that parameter's gradient (the observed error is about
1e-7 of it), plus the bit-identical repeat of a call."""
import numpy as np
import pytest

from oracle import learner as OL
from workload import ActorConfig, EnvConfig, make_actor_weights, make_market, pack_actor_weights

pytestmark = pytest.mark.gpu
NAMES = ("W1", "b1", "W2", "b2", "W3", "b3")


def _rollout(N, D, T, K, H, sigma, key, env_offset, seed, t0=0):
    """T sampled steps from day t0: the first t0 steps run as a separate rollout whose samples are
    dropped, so the kept samples come from a rollout resumed on day t0."""
    import torch
    from paper_2501_10709_amd.vecenv import Ensemble, VecEnv
    cfg = EnvConfig(n_envs=N, n_stocks=D, n_ind=5, n_days=t0 + T)
    m = make_market(seed, D, t0 + T)
    acfg = ActorConfig(n_actors=K, in_dim=cfg.state_dim, hidden=H, out_dim=D, bias_std=0.1, seed_base=300 + seed)
    actors = make_actor_weights(acfg)
    env = VecEnv(cfg, m.close, m.ind, device=torch.device("cuda:0"))
    ens = Ensemble(pack_actor_weights(actors), K, cfg.state_dim, H, D, dtype="f32", max_batch=N)
    s0 = env.reset()
    if t0 > 0:
        first = env.rollout(t0, ens=ens, sigma=sigma, noise_key=key, env_offset=env_offset, path="plain",
                            store=("obs",))
        s0 = first["obs"][-1]
        assert env.day == t0
    out = env.rollout(T, ens=ens, sigma=sigma, noise_key=key, env_offset=env_offset, path="plain", store=("obs", "rew"))
    states = torch.cat([s0[None], out["obs"][:-1]], 0).contiguous()
    return cfg, actors, states, out["rew"].contiguous()


def _unflatten(flat, S, H, A):
    out, o = {}, 0
    for name, shp in (("W1", (S, H)), ("b1", (H,)), ("W2", (H, H)), ("b2", (H,)), ("W3", (H, A)), ("b3", (A,))):
        n = int(np.prod(shp))
        out[name] = flat[o:o + n].reshape(shp)
        o += n
    return out


@pytest.mark.parametrize("agent,lam,N,T,K,H,t0", [(0, 0.0, 24, 16, 3, 64, 0), (2, 0.5, 37, 9, 3, 64, 0),
                                                  (1, 2.0, 130, 5, 3, 64, 0), (0, 1.0, 1, 1, 1, 64, 0),
                                                  (1, 0.3, 50, 7, 3, 128, 0), (2, 0.4, 40, 6, 3, 64, 5)])
def test_policy_gradient_matches_oracle(agent, lam, N, T, K, H, t0):
    """The fourth case is degenerate: one actor (no diversity term whatever lambda), one
    environment, one day.  The fifth has a hidden width of one row tile (128), where the bias
    gradients come from column sums inside the weight-gradient product.  The last takes its
    samples from a rollout resumed on day 5: the regenerated noise must be that of days 5..10."""
    import torch
    from paper_2501_10709_amd import binding as B
    D, sigma, key, off = 5, 0.1, 9, 4
    cfg, actors, states, rew = _rollout(N, D, T, K, H, sigma, key, off, seed=agent + 3, t0=t0)
    S, A = cfg.state_dim, D
    w = torch.as_tensor(pack_actor_weights(actors)).cuda()
    per = S * H + H + H * H + H + H * A + A
    ws = torch.empty(B.fm_pg_workspace_bytes(K, S, H, A, N, T), dtype=torch.uint8, device="cuda")
    g1 = torch.empty(per, dtype=torch.float32, device="cuda")
    g2 = torch.empty_like(g1)
    print(f"policy gradient agent {agent} lambda {lam} N {N} T {T} K {K} H {H} t0 {t0}", flush=True)
    B.fm_policy_gradient(K, S, H, A, w, agent, states, rew, N, T, sigma, key, off, lam, g1, ws, t0=t0)
    B.fm_policy_gradient(K, S, H, A, w, agent, states, rew, N, T, sigma, key, off, lam, g2, ws, t0=t0)
    torch.cuda.synchronize()
    assert torch.equal(g1, g2)
    got = _unflatten(g1.cpu().numpy().astype(np.float64), S, H, A)
    want = OL.policy_gradient(actors, agent, states.cpu().numpy(), rew.cpu().numpy(), sigma, key, off, lam, t0=t0)
    for name in NAMES:
        scale = np.abs(want[name]).max()
        assert scale > 0, name
        err = np.abs(got[name] - want[name]).max()
        print(f"  {name}: max error {err / scale:.2e} of scale", flush=True)
        assert err <= 1e-5 * scale, (name, err, scale)
    if t0 > 0:
        # Keyed by the row index instead of the day, the layer-3 gradient would differ.
        wrong = OL.policy_gradient(actors, agent, states.cpu().numpy(), rew.cpu().numpy(), sigma, key, off, lam)
        assert np.abs(wrong["b3"] - got["b3"]).max() > 1e-3 * np.abs(want["b3"]).max()


def test_policy_gradient_argument_errors():
    import torch
    from paper_2501_10709_amd import binding as B
    K, S, H, A, N, T = 2, 8, 16, 3, 4, 2
    w = torch.zeros(K * (S * H + H + H * H + H + H * A + A), device="cuda")
    st = torch.zeros((T, N, S), device="cuda")
    rw = torch.zeros((T, N), dtype=torch.float64, device="cuda")
    g = torch.zeros(S * H + H + H * H + H + H * A + A, device="cuda")
    ws = torch.empty(B.fm_pg_workspace_bytes(K, S, H, A, N, T), dtype=torch.uint8, device="cuda")
    for kw in (dict(agent=2), dict(sigma=0.0), dict(lam=-1.0), dict(t0=-1)):
        with pytest.raises(B.FmError):
            B.fm_policy_gradient(K, S, H, A, w, kw.get("agent", 0), st, rw, N, T, kw.get("sigma", 0.1), 1, 0,
                                 kw.get("lam", 0.0), g, ws, t0=kw.get("t0", 0))
    small = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(B.FmError):
        B.fm_policy_gradient(K, S, H, A, w, 0, st, rw, N, T, 0.1, 1, 0, 0.0, g, small)


@pytest.mark.parametrize("H,D,N,T", [(32, 3, 3, 2), (96, 33, 65, 3), (160, 10, 33, 4), (300, 40, 20, 9), (256, 31, 9, 257)])
def test_policy_gradient_at_tile_edges(H, D, N, T):
    """Widths on both sides of the tile widths (32, 64, 128, 256) and sums that end inside a block
    of 32 terms; row counts on both sides of a chunk of 2048."""
    import torch
    from paper_2501_10709_amd import binding as B
    S, K, sigma, key = 7 * D + 1, 2, 0.1, 5
    actors = make_actor_weights(ActorConfig(n_actors=K, in_dim=S, hidden=H, out_dim=D, bias_std=0.1, seed_base=77))
    rng = np.random.default_rng(H)
    states = rng.normal(0.0, 0.5, (T, N, S)).astype(np.float32)
    rew = rng.normal(0.0, 1.0, (T, N))
    w = torch.as_tensor(pack_actor_weights(actors)).cuda()
    ws = torch.empty(B.fm_pg_workspace_bytes(K, S, H, D, N, T), dtype=torch.uint8, device="cuda")
    g = torch.empty(S * H + H + H * H + H + H * D + D, dtype=torch.float32, device="cuda")
    B.fm_policy_gradient(K, S, H, D, w, 1, torch.as_tensor(states).cuda(), torch.as_tensor(rew).cuda(), N, T, sigma, key,
                         0, 0.3, g, ws)
    got = _unflatten(g.cpu().numpy().astype(np.float64), S, H, D)
    want = OL.policy_gradient(actors, 1, states, rew, sigma, key, 0, 0.3)
    for name in NAMES:
        scale = np.abs(want[name]).max()
        assert np.abs(got[name] - want[name]).max() <= 1e-5 * scale, name


def test_policy_gradient_with_infinite_and_huge_inputs():
    """An infinite state entry saturates its row's first layer and makes its own weight row's
    gradient infinite or NaN; one beyond the bfloat16 range (3.39e38) is finite.  All other gradients are
    those of float32 arithmetic with the same entries."""
    import torch
    from paper_2501_10709_amd import binding as B
    S, H, D, K, N, T = 8, 64, 3, 1, 40, 3
    per = S * H + H + H * H + H + H * D + D
    g = torch.Generator(device="cuda").manual_seed(3)
    w = torch.randn(per, generator=g, device="cuda") * 0.2
    states = torch.randn((T, N, S), generator=g, device="cuda")
    states[1, 7, 2] = float("inf")
    states[2, 9, 5] = 3.4e38
    rew = torch.randn((T, N), generator=g, device="cuda", dtype=torch.float64)
    ws = torch.empty(B.fm_pg_workspace_bytes(K, S, H, D, N, T), dtype=torch.uint8, device="cuda")
    got = torch.empty(per, device="cuda")
    B.fm_policy_gradient(K, S, H, D, w, 0, states, rew, N, T, 0.1, 1, 0, 0.0, got, ws)
    x = states.reshape(T * N, S).cpu()
    o, p = 0, []
    for shp in ((S, H), (H,), (H, H), (H,), (H, D), (D,)):
        p.append(w[o:o + int(np.prod(shp))].cpu().reshape(shp))
        o += int(np.prod(shp))
    h1 = torch.tanh(x @ p[0] + p[1])
    h2 = torch.tanh(h1 @ p[2] + p[3])
    assert torch.isfinite(h2).all()
    mu = torch.tanh(h2 @ p[4] + p[5])
    eps = torch.empty((T, N, D), device="cuda")
    for t in range(T):
        B.fm_noise(1, 0, N, t, D, eps[t])
    ret = (rew.sum(0) / N).float().cpu().repeat(T)[:, None]
    g3 = ret * (0.1 * eps.reshape(T * N, D).cpu()) / 0.01 * (1 - mu * mu)
    g2 = (g3 @ p[4].t()) * (1 - h2 * h2)
    g1 = (g2 @ p[2].t()) * (1 - h1 * h1)
    want = torch.cat([v.reshape(-1) for v in (x.t() @ g1, g1.sum(0), h1.t() @ g2, g2.sum(0), h2.t() @ g3, g3.sum(0))])
    got = got.cpu()
    row = torch.arange(per) // H
    plain = ~((row == 2) | (row == 5)) | (torch.arange(per) >= S * H)
    assert torch.isfinite(want[plain]).all()
    err = (got - want)[plain].abs().max() / want[plain].abs().max()
    assert err <= 1e-5, err
    assert torch.equal(torch.isfinite(got), torch.isfinite(want))


def _direct(S, H, D, N, T, w, states, rew, sigma, key):
    """One actor's gradient without the library: float64 on the CPU, with the library's noise."""
    import torch
    from paper_2501_10709_amd import binding as B
    o, p = 0, []
    for shp in ((S, H), (H,), (H, H), (H,), (H, D), (D,)):
        p.append(w[o:o + int(np.prod(shp))].cpu().double().reshape(shp))
        o += int(np.prod(shp))
    x = states.reshape(T * N, S).cpu().double()
    h1 = torch.tanh(x @ p[0] + p[1])
    h2 = torch.tanh(h1 @ p[2] + p[3])
    mu = torch.tanh(h2 @ p[4] + p[5])
    eps = torch.empty((T, N, D), device="cuda")
    for t in range(T):
        B.fm_noise(key, 0, N, t, D, eps[t])
    g3 = (rew.sum(0) / N).cpu().repeat(T)[:, None] * eps.reshape(T * N, D).cpu().double() / sigma * (1 - mu * mu)
    g2 = (g3 @ p[4].t()) * (1 - h2 * h2)
    g1 = (g2 @ p[2].t()) * (1 - h1 * h1)
    return (x.t() @ g1, g1.sum(0), h1.t() @ g2, g2.sum(0), h2.t() @ g3, g3.sum(0))


def _one_actor(S, H, D, N, T, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.randn(S * H + H + H * H + H + H * D + D, generator=g, device="cuda") * 0.2
    states = torch.randn((T, N, S), generator=g, device="cuda")
    rew = torch.randn((T, N), generator=g, device="cuda", dtype=torch.float64)
    return w, states, rew


def _gradient(S, H, D, N, T, w, states, rew, sigma, key):
    import torch
    from paper_2501_10709_amd import binding as B
    ws = torch.empty(B.fm_pg_workspace_bytes(1, S, H, D, N, T), dtype=torch.uint8, device="cuda")
    got = torch.empty(S * H + H + H * H + H + H * D + D, device="cuda")
    call = lambda: B.fm_policy_gradient(1, S, H, D, w, 0, states, rew, N, T, sigma, key, 0, 0.0, got, ws)  # noqa: E731
    call()
    return got, call


@pytest.mark.parametrize("S,H,D,N,T", [(9, 32, 3, 41, 3), (36, 64, 33, 9, 7), (33, 96, 5, 700, 3), (20, 128, 40, 77, 4),
                                       (50, 300, 31, 50, 5), (128, 256, 66, 65, 2)])
def test_policy_gradient_past_the_bfloat16_range(S, H, D, N, T):
    """Operands that have no bfloat16 value (an infinite state entry; weights of 3.4e38 in layers 2 and
    3, whose units saturate) on every layout and tile width of the products, with remainders in rows,
    columns and terms: all entries that are finite are the gradient's."""
    import torch
    w, states, rew = _one_actor(S, H, D, N, T, 11)
    states[1, 7, 2] = float("inf")
    w[S * H + H + 3 * H + 5] = 3.4e38
    w[S * H + H + H * H + H + 4 * D + 1] = -3.4e38
    got, _ = _gradient(S, H, D, N, T, w, states, rew, 0.1, 1)
    got = _unflatten(got.cpu().double(), S, H, D)
    for name, want in zip(NAMES, _direct(S, H, D, N, T, w, states, rew, 0.1, 1)):
        if name == "W1":
            keep = torch.arange(S) != 2
            got[name], want = got[name][keep], want[keep]
        assert torch.isfinite(want).all() and torch.isfinite(got[name]).all(), name
        err = (got[name] - want).abs().max() / want.abs().max()
        assert err <= 1e-5, (name, err)


def test_policy_gradient_time_with_a_nan_reward():
    """One NaN reward makes every entry of the gradient NaN.  It costs a second pass of the products
    in float32 (about twice the time), and not one element at a time (over a hundred times)."""
    import torch
    S, H, D, N, T = 211, 256, 30, 1000, 20
    w, states, rew = _one_actor(S, H, D, N, T, 5)

    def ms(call):
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            call()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return sorted(times)[2]

    got, call = _gradient(S, H, D, N, T, w, states, rew, 0.1, 1)
    assert torch.isfinite(got).all()
    plain = ms(call)
    rew[3, 500] = float("nan")
    got, call = _gradient(S, H, D, N, T, w, states, rew, 0.1, 1)
    assert torch.isnan(got).all()
    nan = ms(call)
    print(f"  finite {plain:.3f} ms, one NaN reward {nan:.3f} ms", flush=True)
    assert nan <= 10 * plain, (nan, plain)


@pytest.mark.parametrize("reward,column,weight", [(1e-36, 1.0, 1.0), (1.0, 1e-36, 1.0), (1.0, 1e-34, 1e34), (1e25, 1.0, 1.0),
                                                  (1e30, 1.0, 1.0)])
def test_policy_gradient_at_the_ends_of_the_float32_range(reward, column, weight):
    """Rewards, and one state column with its weights, at magnitudes where a part of a split operand
    leaves the bfloat16 range or a scaled sum the float32 one; each row of a matrix is held to its own
    largest entry.  (Rewards of 1e-37 make subnormal deltas, of fewer bits in float32 itself.)"""
    import torch
    S, H, D, N, T = 40, 96, 7, 200, 12
    w, states, rew = _one_actor(S, H, D, N, T, 21)
    rew *= reward
    states[:, :, 3] *= column
    w[3 * H:4 * H] *= weight
    got, _ = _gradient(S, H, D, N, T, w, states, rew, 0.1, 1)
    got = _unflatten(got.cpu().double(), S, H, D)
    for name, want in zip(NAMES, _direct(S, H, D, N, T, w, states, rew, 0.1, 1)):
        scale = want.abs().amax(-1, keepdim=True)
        err = ((got[name] - want).abs() / scale).max()
        print(f"  {name}: largest {scale.max():.1e}, error {err:.1e}", flush=True)
        assert err <= 1e-5, (name, err)
