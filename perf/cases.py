"""The work that users of the trading-environment library have it do, as timed cases.

A case is a dict of plain values; `prepare` makes what a program holds before the call, `run` is
one pass through the public entry points, `work` what that pass cannot do without and `exact` its
outputs in 64-bit arithmetic where they are computed numbers.  Kinds of case:

  steps   an episode driven from Python, one VecEnv.step per day
  driven  VecEnv.rollout over given actions (a backtest; with `metrics` also its evaluation)
  plain   the closed-loop float32 rollout (ensemble and environment launched per day)
  fused   the closed-loop bfloat16 rollout (sampling for training)
  act     Ensemble.act on a batch of states (policy inference outside a rollout)
  batch   uneven groups of environments run as one job
  serve   crypto requests submitted to the continuous-batching server and run to the end
  learn   one policy gradient from a stored rollout
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2501_10709_amd import binding as B
from paper_2501_10709_amd.serve import CryptoServer
from paper_2501_10709_amd.vecenv import Batch, Ensemble, VecEnv

IND = 5          # indicators per stock
SIGMA = 0.1      # exploration noise
BIAS_STD = 0.05  # trained actors have biases
HMAX, COST, CASH0, SCALE = 100, 1e-3, 1e6, 2.0 ** -12
TICKS = 200_000  # the crypto tick table
CRYPTO_H = 128


def listed():
    return [
        # The smallest use: a gym-style loop over a handful of environments, one call per day.
        {"name": "steps-16x30", "kind": "steps", "N": 16, "D": 30, "T": 30},
        # Policy inference for a few live portfolios in the deployed precision.
        {"name": "act-bf16-64", "kind": "act", "N": 64, "D": 30, "H": 256, "K": 3, "dtype": "bf16"},
        # Policy inference for a whole vectorised environment in float32.
        {"name": "act-f32-2048", "kind": "act", "N": 2048, "D": 30, "H": 256, "K": 3, "dtype": "f32"},
        # A one-year backtest of given actions at the paper's largest environment count.
        {"name": "driven-2048x252", "kind": "driven", "N": 2048, "D": 30, "T": 252, "metrics": True},
        # Enough environments to fill the GPU many times over.
        {"name": "driven-65536x64", "kind": "driven", "N": 65536, "D": 30, "T": 64, "metrics": False},
        # The float32 closed loop at paper scale.
        {"name": "plain-2048x252", "kind": "plain", "N": 2048, "D": 30, "T": 252, "H": 256, "K": 3},
        # The headline: bfloat16 sampling at paper scale.
        {"name": "fused-2048x252", "kind": "fused", "N": 2048, "D": 30, "T": 252, "H": 256, "K": 3},
        # The same actors on four times as many environments.
        {"name": "fused-8192x252", "kind": "fused", "N": 8192, "D": 30, "T": 252, "H": 256, "K": 3},
        # A portfolio and network size of a user's own: odd stock and environment counts.
        {"name": "fused-1000x100-d17", "kind": "fused", "N": 1000, "D": 17, "T": 100, "H": 128, "K": 3},
        # Groups with their own stock counts, environment counts and horizons, as one job.
        {"name": "batch-24", "kind": "batch", "G": 24, "layout": 4, "n_max": 4096, "t_max": 400},
        # Crypto requests of mixed sizes served together.
        {"name": "serve-24", "kind": "serve", "R": 24, "layout": 5, "n_max": 4096, "h_max": 4096, "K": 5,
         "tile_rows": 64},
        # One gradient from a paper-scale rollout.
        {"name": "learn-2048x252", "kind": "learn", "N": 2048, "D": 30, "T": 252, "H": 256, "K": 3},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["steps", "act", "driven", "plain", "fused", "fused", "batch", "serve", "learn"])
    if kind == "steps":
        return {"kind": kind, "N": _log_int(rng, 1, 4096), "D": rng.randint(3, 32), "T": rng.randint(5, 50)}
    if kind == "act":
        return {"kind": kind, "N": _log_int(rng, 1, 8192), "D": rng.randint(3, 50), "H": rng.choice([64, 128, 256]),
                "K": rng.choice([1, 3, 5]), "dtype": rng.choice(["f32", "bf16"])}
    if kind == "driven":
        n = _log_int(rng, 16, 65536)
        return {"kind": kind, "N": n, "D": rng.randint(3, 32), "T": max(5, min(252, 4_000_000 // n)),
                "metrics": rng.random() < 0.5}
    if kind == "plain":
        return {"kind": kind, "N": _log_int(rng, 16, 2048), "D": rng.randint(3, 32), "T": rng.randint(10, 252),
                "H": rng.choice([64, 128, 256]), "K": rng.choice([1, 3])}
    if kind == "fused":
        # Two in three are the trading year of 30 stocks at some environment count; the others
        # have a shape of their own.
        if rng.random() < 0.67:
            return {"kind": kind, "N": _log_int(rng, 16, 8192), "D": 30, "T": rng.randint(10, 252), "H": 256, "K": 3}
        return {"kind": kind, "N": _log_int(rng, 16, 4096), "D": rng.randint(3, 60), "T": rng.randint(10, 126),
                "H": rng.choice([64, 128, 256]), "K": rng.choice([1, 3])}
    if kind == "batch":
        return {"kind": kind, "G": rng.randint(2, 24), "layout": rng.randint(10, 10_000),
                "n_max": _log_int(rng, 64, 4096), "t_max": rng.randint(30, 400)}
    if kind == "serve":
        return {"kind": kind, "R": rng.randint(1, 24), "layout": rng.randint(10, 10_000),
                "n_max": _log_int(rng, 16, 4096), "h_max": rng.randint(300, 4096), "K": rng.choice([1, 3, 5]),
                "tile_rows": rng.choice([16, 64])}
    n = _log_int(rng, 16, 2048)
    return {"kind": kind, "N": n, "D": rng.randint(3, 40), "T": rng.randint(10, 252), "H": rng.choice([64, 128, 256]),
            "K": rng.choice([1, 3])}


# ------------------------------------------------------------------------------------------------
# Inputs
# ------------------------------------------------------------------------------------------------

def _width(D):
    return (IND + 2) * D + 1


def _config(N, D, T):
    return SimpleNamespace(n_envs=N, n_stocks=D, n_ind=IND, n_days=T, hmax=HMAX, init_cash=CASH0, cost_rate=COST,
                           reward_scale=SCALE, cash_obs_scale=2.0 ** -20, price_obs_scale=2.0 ** -8,
                           hold_obs_scale=2.0 ** -10)


def _market(rng, D, T, vol=0.02):
    """Daily closes [T+1][D] of a geometric Brownian motion and indicators [T+1][IND][D]."""
    z = rng.standard_normal((T + 1, D))
    close = rng.uniform(50, 300, D) * np.exp(np.cumsum(3e-4 - vol * vol / 2 + vol * z, axis=0))
    width = np.array([0.02, 0.04, 0.15, 0.3, 0.02])[:, None]
    ind = rng.standard_normal((T + 1, IND, D)) * width
    return close.astype(np.float32), ind.astype(np.float32)


def _weights(rng, K, S, H, A, gain=1.0):
    """K actors, Xavier-uniform weights and small biases, in the packed layout."""
    parts = []
    for _ in range(K):
        for i, o, g in ((S, H, 1.0), (H, H, 1.0), (H, A, gain)):
            lim = math.sqrt(6.0 / (i + o))
            parts += [(rng.uniform(-lim, lim, i * o) * g).astype(np.float32),
                      (rng.standard_normal(o) * BIAS_STD).astype(np.float32)]
    return np.concatenate(parts)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _actions(seed, T, N, D):
    """Actions in [-1, 1], leaning towards buying, with zeros, sub-share values and both ends."""
    g = _gen(seed)
    a = torch.rand((T, N, D), generator=g, device="cuda").mul_(2).sub_(0.85)
    u = torch.rand((T, N, D), generator=g, device="cuda")
    a[u < 0.05] = 0.0
    a = torch.where((u >= 0.05) & (u < 0.10), a * 0.0099, a)
    a[(u >= 0.10) & (u < 0.12)] = 1.0
    a[(u >= 0.12) & (u < 0.14)] = -1.0
    return a.clamp_(-1, 1).contiguous()


def _states(seed, T, N, D):
    """Trading states [T][N][S]: own cash and holdings, the day's prices and indicators shared."""
    g = _gen(seed)
    rnd = lambda *s: torch.rand(s, generator=g, device="cuda")  # noqa: E731
    x = torch.empty((T, N, _width(D)), device="cuda")
    x[..., 0] = rnd(T, N)
    x[..., 1:1 + D] = (50 + 250 * rnd(T, 1, D)) * 2.0 ** -8
    x[..., 1 + D:1 + 2 * D] = (300 * rnd(T, N, D)).floor() * 2.0 ** -10
    x[..., 1 + 2 * D:] = 0.1 * torch.randn((T, 1, IND * D), generator=g, device="cuda")
    return x


def _groups(case):
    """Sizes of an uneven batch: stock counts from a few index sizes, environment counts log-uniform."""
    r = np.random.default_rng(case["layout"])
    return [(int(math.exp(r.uniform(math.log(32), math.log(case["n_max"])))), int(r.choice([5, 10, 30, 50, 100])),
             int(r.integers(20, case["t_max"] + 1)), float(r.uniform(0.01, 0.04))) for _ in range(case["G"])]


def _requests(case):
    """(environments, horizon) of each crypto request, log-uniform."""
    r = np.random.default_rng(case["layout"])
    return [(int(math.exp(r.uniform(0, math.log(case["n_max"])))),
             int(math.exp(r.uniform(math.log(200), math.log(case["h_max"]))))) for _ in range(case["R"])]


def _ticks(rng):
    """Mid prices and the 16-column feature table (columns 3..15) of a heavy-tailed tick series."""
    r = rng.standard_t(3, size=TICKS) / math.sqrt(3.0) * 1e-4
    feat = np.zeros((TICKS, 16), np.float32)
    for i in range(10):
        feat[i:, 3 + i] = r[:TICKS - i] * 1e4
    feat[:, 13:15] = np.abs(rng.standard_normal((TICKS, 2)))
    feat[:, 15] = rng.uniform(-1, 1, TICKS)
    return 50_000.0 * np.exp(np.cumsum(r)), feat


def prepare(case, seed):
    kind, rng = case["kind"], np.random.default_rng(seed)
    s = SimpleNamespace(case=case, kind=kind, out=None, key=1 + seed % 1_000_003)
    if kind in ("steps", "driven", "plain", "fused"):
        N, D, T = case["N"], case["D"], case["T"]
        s.env = VecEnv(_config(N, D, T), *_market(rng, D, T))
        if kind in ("steps", "driven"):
            s.actions = _actions(seed, T, N, D)
        else:
            s.ens = Ensemble(_weights(rng, case["K"], _width(D), case["H"], D), case["K"], _width(D), case["H"], D,
                             dtype="f32" if kind == "plain" else "bf16", max_batch=N)
    elif kind == "act":
        D, S = case["D"], _width(case["D"])
        s.ens = Ensemble(_weights(rng, case["K"], S, case["H"], D), case["K"], S, case["H"], D, dtype=case["dtype"],
                         max_batch=case["N"])
        s.obs = _states(seed, 1, case["N"], D)[0].contiguous()
    elif kind == "batch":
        s.envs, spec = [], []
        for i, (N, D, T, vol) in enumerate(_groups(case)):
            env = VecEnv(_config(N, D, T), *_market(rng, D, T, vol))
            ens = Ensemble(_weights(rng, 3, _width(D), 256, D), 3, _width(D), 256, D, dtype="bf16", max_batch=N)
            env.reset(return_obs=False)
            s.envs.append((env, ens))
            spec.append(dict(env=env, ens=ens, n_steps=T, sigma=SIGMA, noise_key=s.key, env_offset=4096 * i,
                             store=("act", "rew")))
        s.batch = Batch(spec)
        s.batch.tune()
        for env, _ in s.envs:
            env.reset(return_obs=False)
    elif kind == "serve":
        mid, feat = _ticks(rng)
        s.srv = CryptoServer(mid, feat, _weights(rng, case["K"], 16, CRYPTO_H, 3, gain=4.0), case["K"], eps=0.005,
                             fee=2e-4, tile_rows=case["tile_rows"], chunk_ticks=256)
        s.reqs = []
        for n, h in _requests(case):
            stride = int(rng.integers(0, min(40, (TICKS - h - 200) // max(1, n)) + 1))
            start = 64 + int(rng.integers(0, TICKS - 65 - h - stride * (n - 1)))
            s.reqs.append((n, h, start, stride, int(rng.integers(1, 1 << 40))))
    else:
        N, D, T, H, K = case["N"], case["D"], case["T"], case["H"], case["K"]
        S = _width(D)
        s.w = torch.from_numpy(_weights(rng, K, S, H, D)).cuda()
        s.states = _states(seed, T, N, D)
        s.rew = 2.0 * torch.randn((T, N), generator=_gen(seed + 1), device="cuda", dtype=torch.float64)
        s.grad = torch.empty(S * H + H + H * H + H + H * D + D, device="cuda")
        s.ws = torch.empty(B.fm_pg_workspace_bytes(K, S, H, D, N, T), dtype=torch.uint8, device="cuda")
    return s


# ------------------------------------------------------------------------------------------------
# One pass
# ------------------------------------------------------------------------------------------------

def run(s):
    c = s.case
    if s.kind == "steps":
        obs, rews, qty = s.env.reset(), [], None
        for t in range(c["T"]):
            obs, rew, qty, done = s.env.step(s.actions[t])
            rews.append(rew)
        return {"obs": obs, "qty": qty, "rew": rews}
    if s.kind == "driven":
        s.env.reset(return_obs=False)
        s.out = s.env.rollout(c["T"], actions=s.actions, store=("obs", "rew", "qty"), out=s.out)
        if not c["metrics"]:
            return dict(s.out)
        return {**s.out, "metrics": B.fm_backtest_metrics(s.out["rew"], CASH0, SCALE)}
    if s.kind in ("plain", "fused"):
        s0 = s.env.reset()
        s.out = s.env.rollout(c["T"], ens=s.ens, sigma=SIGMA, noise_key=s.key, path=s.kind, store=("obs", "act", "rew"),
                              out=s.out)
        return {"s0": s0, **s.out}
    if s.kind == "act":
        act, mean = s.ens.act(s.obs, t=3, sigma=SIGMA, noise_key=s.key, return_mean=True)
        return {"act": act, "mean": mean}
    if s.kind == "batch":
        for env, _ in s.envs:
            env.reset(return_obs=False)
        return list(s.batch.run(use_graph=True))
    if s.kind == "serve":
        ids = [s.srv.submit(n, h, start, stride, key) for n, h, start, stride, key in s.reqs]
        s.srv.run_all()
        out = []
        for rid in ids:
            res = s.srv.result(rid)[0]
            out.append([res.view(np.float64).reshape(-1, 8)[:, :6], res.view(np.int32).reshape(-1, 16)[:, 12:]])
        return out
    B.fm_policy_gradient(c["K"], _width(c["D"]), c["H"], c["D"], s.w, 0, s.states, s.rew, c["N"], c["T"], SIGMA, s.key,
                         0, 0.1, s.grad, s.ws)
    return s.grad


# ------------------------------------------------------------------------------------------------
# What a pass cannot do without
# ------------------------------------------------------------------------------------------------

def _mlp(S, H, A):
    return S * H + H * H + H * A


def work(case):
    kind = case["kind"]
    if kind == "batch":
        b = f = 0
        for N, D, T, _ in _groups(case):
            S = _width(D)
            f += 2 * 3 * _mlp(S, 256, D) * N * T
            b += (4 * D + 8) * N * T + 2 * 3 * _mlp(S, 256, D) + 4 * (T + 1) * (1 + IND) * D
        return {"bytes": b, "flops": f}
    if kind == "serve":
        r = _requests(case)
        return {"bytes": sum(64 * n for n, _ in r) + TICKS * 72,
                "flops": 2 * case["K"] * _mlp(16, CRYPTO_H, 3) * sum(n * h for n, h in r)}
    N, D = case["N"], case["D"]
    S = _width(D)
    if kind in ("steps", "driven"):
        # Per environment and day: the action in; the state, reward and quantities out.  The trades
        # and the value are about 30 operations a stock.
        n = N * case["T"]
        wanted = (4 * S + 4 * D) * (N if kind == "steps" else n) + 8 * n
        return {"bytes": 4 * D * n + wanted + (96 * N if case.get("metrics") else 0), "flops": 30 * D * n}
    H, K = case["H"], case["K"]
    if kind == "act":
        es = 2 if case["dtype"] == "bf16" else 4
        return {"bytes": N * 4 * (S + 2 * D) + K * es * _mlp(S, H, D), "flops": 2 * K * _mlp(S, H, D) * N}
    rows = N * case["T"]
    if kind == "learn":
        return {"bytes": rows * (4 * S + 8) + 4 * (K + 1) * _mlp(S, H, D),
                "flops": rows * (2 * (K + 1) * _mlp(S, H, D) + 2 * (D * H + H * H))}
    es = 2 if kind == "fused" else 4
    return {"bytes": rows * (4 * S + 4 * D + 8) + K * es * _mlp(S, H, D), "flops": rows * 2 * K * _mlp(S, H, D)}


# ------------------------------------------------------------------------------------------------
# The outputs in 64-bit arithmetic.  None where an output is a long closed loop: there a rounding
# that moves one order by one share changes all that follows.
# ------------------------------------------------------------------------------------------------

def _simulate(case, seed):
    """The trading days over given actions (sells, then buys, in stock order) in float64."""
    N, D, T = case["N"], case["D"], case["T"]
    close, ind = (torch.from_numpy(x).cuda().double() for x in _market(np.random.default_rng(seed), D, T))
    act = _actions(seed, T, N, D)
    cash = torch.full((N,), CASH0, device="cuda", dtype=torch.float64)
    hold = torch.zeros((D, N), device="cuda", dtype=torch.float64)
    value = cash.clone()
    keep = case["kind"] == "driven"
    obs = torch.empty((T if keep else 1, N, _width(D)), device="cuda", dtype=torch.float64)
    qty = torch.empty((T if keep else 1, N, D), device="cuda", dtype=torch.int32)
    rew = torch.empty((T, N), device="cuda", dtype=torch.float64)
    for t in range(T):
        q = (act[t] * float(HMAX)).trunc().t().double().contiguous()
        price = close[t].tolist()
        sold = torch.minimum(hold, (-q).clamp_min_(0))
        buy = q.clamp_min(0)
        fill = torch.zeros_like(buy)
        for d in range(D):
            cash = cash + (price[d] * sold[d]) * (1.0 - COST)
        for d in range(D):
            k = torch.minimum(torch.floor(cash / (price[d] * (1.0 + COST))) + 1, buy[d])
            for _ in range(2):
                k = k - ((price[d] * k) * (1.0 + COST) > cash).double()
            fill[d] = k
            cash = cash - (price[d] * k) * (1.0 + COST)
        hold = hold - sold + fill
        new = cash
        for d, p in enumerate(close[t + 1].tolist()):
            new = new + p * hold[d]
        rew[t], value = (new - value) * SCALE, new
        o = obs[t if keep else 0]
        o[:, 0] = cash * 2.0 ** -20
        o[:, 1:1 + D] = close[t + 1] * 2.0 ** -8
        o[:, 1 + D:1 + 2 * D] = hold.t() * 2.0 ** -10
        o[:, 1 + 2 * D:] = ind[t + 1].reshape(-1)
        qty[t if keep else 0] = (fill - sold).t().int()
    if not keep:
        return {"obs": obs[0], "qty": qty[0], "rew": list(rew)}
    out = {"obs": obs, "rew": rew, "qty": qty}
    if case["metrics"]:
        out["metrics"] = _metrics(rew)
    return out


def _metrics(rew):
    v = torch.cat([torch.full_like(rew[:1], CASH0), CASH0 + torch.cumsum(rew / SCALE, 0)], 0)
    rho = v[1:] / v[:-1] - 1
    T, P = rho.shape[0], 252.0
    total = v[-1] / v[0] - 1
    annual = (v[-1] / v[0]) ** (P / T) - 1
    mean, sd = rho.mean(0), rho.std(0)
    mdd = (v / torch.cummax(v, 0).values - 1).min(0).values
    down = rho.clamp_max(0).square().mean(0).sqrt()
    return torch.stack([total, annual, sd * P ** 0.5, mean / sd * P ** 0.5, mdd, total / mdd.abs(),
                        mean / down * P ** 0.5, annual / mdd.abs(), rho.clamp_min(0).sum(0) / (-rho).clamp_min(0).sum(0),
                        (rho > 0).sum(0).double() / (rho < 0).sum(0).double()], 1)


def _noise(key, N, days, D):
    """Standard normals [days][N][D] of the library's counter-based generator, in float64."""
    G = (D + 3) // 4
    w = np.empty((len(days), G, N, 4), np.uint64)
    for i, t in enumerate(days):
        for j in range(G):
            # numpy steps the counter before each block, so it starts one below environment 0.
            counter = (j << 128 | t << 64) - 1
            w[i, j] = np.random.Philox(counter=counter % (1 << 256), key=key).random_raw(4 * N).reshape(N, 4)
    u = ((w >> np.uint64(41)).astype(np.float64) + 0.5) * 2.0 ** -23
    u = torch.from_numpy(u).cuda()
    r0, r1 = (-2 * u[..., 0].log()).sqrt(), (-2 * u[..., 2].log()).sqrt()
    a0, a1 = 2 * math.pi * u[..., 1], 2 * math.pi * u[..., 3]
    z = torch.stack([r0 * a0.cos(), r0 * a0.sin(), r1 * a1.cos(), r1 * a1.sin()], -1)
    return z.permute(0, 2, 1, 3).reshape(len(days), N, 4 * G)[..., :D]


def _actor(w, k, S, H, A, bf16=False):
    """Float64 matrices and biases of actor k from the packed weights."""
    sizes = [(S, H), (H,), (H, H), (H,), (H, A), (A,)]
    o, p = k * sum(math.prod(x) for x in sizes), []
    for shape in sizes:
        x = w[o:o + math.prod(shape)].reshape(shape)
        p.append((x.bfloat16() if bf16 and len(shape) == 2 else x).double())
        o += math.prod(shape)
    return p


def _forward(p, x):
    h1 = torch.tanh(x @ p[0] + p[1])
    h2 = torch.tanh(h1 @ p[2] + p[3])
    return h1, h2, torch.tanh(h2 @ p[4] + p[5])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("steps", "driven"):
        return _simulate(case, seed)
    if kind not in ("act", "learn"):
        return None
    N, D, H, K = case["N"], case["D"], case["H"], case["K"]
    S, key = _width(D), 1 + seed % 1_000_003
    w = torch.from_numpy(_weights(np.random.default_rng(seed), K, S, H, D)).cuda()
    if kind == "act":
        x = _states(seed, 1, N, D)[0].double()
        mean = sum(_forward(_actor(w, k, S, H, D, case["dtype"] == "bf16"), x)[2] for k in range(K)) / K
        return {"act": (mean + SIGMA * _noise(key, N, [3], D)[0]).clamp(-1, 1), "mean": mean}
    T = case["T"]
    x = _states(seed, T, N, D).reshape(T * N, S).double()
    rew = 2.0 * torch.randn((T, N), generator=_gen(seed + 1), device="cuda", dtype=torch.float64)
    mine = _actor(w, 0, S, H, D)
    h1, h2, mu = _forward(mine, x)
    mean, div = mu / K, torch.zeros_like(mu)
    for k in range(1, K):
        other = _forward(_actor(w, k, S, H, D), x)[2]
        mean, div = mean + other / K, div + (mu - other)
    a = mean + SIGMA * _noise(key, N, range(T), D).reshape(T * N, D)
    u = (rew.sum(0) / N).repeat(T)[:, None] * (a - mu) / SIGMA ** 2 + 0.1 / (N * T) * div / SIGMA ** 2
    g3 = u * (1 - mu * mu)
    g2 = (g3 @ mine[4].t()) * (1 - h2 * h2)
    g1 = (g2 @ mine[2].t()) * (1 - h1 * h1)
    return torch.cat([v.reshape(-1) for v in (x.t() @ g1, g1.sum(0), h1.t() @ g2, g2.sum(0), h2.t() @ g3, g3.sum(0))])
