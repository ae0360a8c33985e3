"""Rollout inference of networks outside the general fused block: narrow ones
(two waves), wide ones (the tiled first layer) and observation widths that are
no multiple of 16, at block edges, against the layer-by-layer kernels (which
the parity tests hold to the oracle).  The hidden layers of both paths round
alike, so the means and values may differ by the output layer's float32
summation alone (1e-5, the float32 tolerance) and the log-densities not at
all; those are checked against the oracle too."""
import numpy as np
import pytest
import torch

import paper_2109_11978_amd as ppo
import synth
from oracle import NetSpec, rollout_infer
from tests.gpu_common import dev, require_gpu
from tests.parity import TOL, assert_close

pytestmark = pytest.mark.gpu

# (obs dim, actions, hidden widths, environments)
NARROW = [(48, 12, (64, 64), 64), (45, 10, (64,), 1), (235, 4, (256, 128, 64), 33), (7, 16, (64, 256, 128, 64), 31),
          (33, 12, (128, 64), 97)]
WIDE = [(235, 12, (1024, 512, 256), 65), (48, 8, (1024, 512, 256), 1), (225, 16, (768, 256, 128), 130),
        (256, 2, (512, 512, 512), 63), (17, 12, (1024, 512), 64), (100, 6, (256, 512, 256, 512), 200),
        (300, 12, (1024, 512, 256), 65), (500, 8, (768, 256, 128), 31)]   # inputs past the last tile
ODD = [(225, 12, (512, 256, 128), 100), (5, 12, (128, 128), 32), (57, 14, (256, 128), 40)]


def infer(net, theta, obs, device, fused, monkeypatch, value_only=False):
    monkeypatch.setenv("PPO_FUSED", "1" if fused else "0")
    D, A, H = net
    N = obs.shape[0]
    ctx = ppo.Context(D, A, H, "bf16")
    params = ppo.Params(ctx, theta, device=device)
    out = dict(values=torch.full((N,), float("nan"), device=device))
    if not value_only:
        out.update(actions=torch.full((N, A), float("nan"), device=device),
                   logp=torch.full((N,), float("nan"), device=device),
                   mu=torch.full((N, A), float("nan"), device=device))
    ws = ctx.new_workspace(N=N)
    ws.fill_(0xFF)   # NaN everywhere: nothing unwritten may be read
    ppo.ppo_rollout_infer(ctx, params, dev(obs, device), t=3, seed=11, iteration=2, ws=ws, **out)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("D,A,H,N", NARROW + WIDE + ODD)
def test_infer_shapes(D, A, H, N, monkeypatch):
    d = require_gpu()
    print(f"[gpu-case] infer D={D} A={A} H={H} N={N}", flush=True)
    net = synth.NetShape(D, A, H)
    theta = synth.xavier_theta(net, seed=3, logstd=-0.25)
    theta += 0.02 * np.random.default_rng(1).standard_normal(theta.shape).astype(np.float32)
    obs = synth.rollout.gaussian_like((N, D), seed=5)
    got = infer((D, A, H), theta, obs, d, True, monkeypatch)
    layered = infer((D, A, H), theta, obs, d, False, monkeypatch)
    ref = rollout_infer(theta, NetSpec(D, A, H), obs, seed=11, t=3, iteration=2)
    for k in ("mu", "values", "actions"):
        assert_close(k, got[k], layered[k].astype(np.float64), TOL["fp32"])
    assert np.array_equal(got["logp"], layered["logp"])
    assert_close("logp", got["logp"], ref["logp"], TOL["fp32"])
    only = infer((D, A, H), theta, obs, d, True, monkeypatch, value_only=True)
    assert np.array_equal(only["values"], got["values"])


@pytest.mark.parametrize("D,A,H", [(48, 12, (64, 64)), (235, 12, (1024, 512, 256)), (5, 12, (128, 128))])
def test_tuning_answers_without_tiles(D, A, H):
    """The tile query works after inference of a network for which
    fused_infer_shape reports no fused block, and not before."""
    d = require_gpu()
    net = synth.NetShape(D, A, H)
    ctx = ppo.Context(D, A, H, "bf16")
    assert ctx.fused_infer_shape() == (0, 0)
    params = ppo.Params(ctx, synth.xavier_theta(net, seed=3, logstd=-0.25), device=d)
    with pytest.raises(ppo.PPOError):
        ctx.tuning(40, False)
    ppo.ppo_rollout_infer(ctx, params, dev(synth.rollout.gaussian_like((40, D), seed=5), d), t=0, seed=1,
                          iteration=0, ws=ctx.new_workspace(N=40), values=torch.empty(40, device=d))
    assert set(ctx.tuning(40, False)) == {f"forward_{l + 1}" for l in range(len(H))}
    with pytest.raises(ppo.PPOError):
        ctx.tuning(41, False)
