"""The ensemble MLP at the edges of its tiles: batches around one and two row tiles and past the
size where the tiles widen, hidden widths below, at and past one output tile per wavefront, odd
state widths, and output widths with and without a split of the last layer -- against the oracle."""
import numpy as np
import pytest

from _helpers import TOL_BF16, TOL_F32, actors_case, cuda
from oracle.policy import device_weights, ensemble_mean

pytestmark = pytest.mark.gpu

# n, S, H, A, K
SHAPES = [(1, 1, 32, 1, 1), (16, 211, 64, 30, 3), (17, 33, 288, 17, 2), (33, 255, 256, 128, 3), (1367, 211, 256, 30, 3),
          (40, 700, 512, 48, 2)]


@pytest.mark.parametrize("dtype,tol", [("f32", TOL_F32), ("bf16", TOL_BF16)])
@pytest.mark.parametrize("n,S,H,A,K", SHAPES)
def test_mlp_at_tile_edges(n, S, H, A, K, dtype, tol):
    import torch
    from paper_2501_10709_amd.vecenv import Ensemble
    dev = cuda()
    obs = np.random.default_rng(7).standard_normal((n, S)).astype(np.float32)
    acfg, actors, packed = actors_case(K, S, H, A)
    ens = Ensemble(packed, K, S, H, A, dtype=dtype, max_batch=n, device=dev)
    _, mean = ens.act(torch.from_numpy(obs).to(dev), t=0, sigma=0.0, return_mean=True)
    ref = ensemble_mean(device_weights(actors, dtype), obs)
    assert np.abs(mean.cpu().numpy() - ref).max() <= tol


@pytest.mark.parametrize("S,H,ok", [(736, 512, True), (737, 512, False), (1024, 256, False), (1024, 224, True)])
def test_float32_width_limit_past_16_rows(S, H, ok):
    """State width (rounded up to 32) and hidden width together reach 1280: 16 rows a call are taken, 17
    refused, and the refusal leaves nothing behind for the next call."""
    import torch
    from paper_2501_10709_amd import binding as B
    from paper_2501_10709_amd.vecenv import Ensemble
    dev = cuda()
    acfg, actors, packed = actors_case(1, S, H, 5)
    obs = np.random.default_rng(3).standard_normal((17, S)).astype(np.float32)
    d_obs = torch.from_numpy(obs).to(dev)
    ens = Ensemble(packed, 1, S, H, 5, dtype="f32", max_batch=17, device=dev)
    if not ok:
        with pytest.raises(B.FmError):
            ens.act(d_obs, t=0)
    n = 17 if ok else 16
    _, mean = ens.act(d_obs[:n], t=0, sigma=0.0, return_mean=True)
    ref = ensemble_mean(device_weights(actors, "f32"), obs[:n])
    assert np.abs(mean.cpu().numpy() - ref).max() <= TOL_F32
