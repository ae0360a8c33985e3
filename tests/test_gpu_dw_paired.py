"""Weight gradients in 256 x 128 tiles (wide networks, bf16) at the edges of
their split over the samples, against the gradient with 64 x 128 tiles and
another split count.  Both read the same bf16 operands (the fused pass's), so
they differ by float32 accumulation alone: each is within 8 ulps sqrt(rows) of
the exact sums (the GEMM tests' bound), relative to the rms of the layer's
gradient (a bias is the weight of an input of one)."""
import numpy as np
import pytest
import torch

import paper_2109_11978_amd as ppo
import synth
from oracle import NetSpec, param_layout
from tests.gpu_common import dev, require_gpu, teacher_batch

pytestmark = pytest.mark.gpu


def gradient(D, A, H, theta, batch, M, dw_tile, d, monkeypatch, tmp_path):
    # the tuning file fixes the weight gradient's tile (the last site)
    path = tmp_path / f"tune{dw_tile}"
    path.write_text(f"bf16|{D}|{A}|{''.join(f'{h},' for h in H)}|{M}|u|2{' 0 2' * 8} {dw_tile} 2\n")
    monkeypatch.setenv("PPO_TUNE_CACHE", str(path))
    monkeypatch.delenv("PPO_AUTOTUNE", raising=False)
    ctx = ppo.Context(D, A, H, "bf16")
    params = ppo.Params(ctx, theta, device=d)
    stats = torch.zeros(ppo.PPO_STATS_WIDTH, device=d)
    ws = ctx.new_workspace(M=M)
    ws.fill_(0xFF)   # NaN everywhere: nothing unwritten may be read
    grad = torch.full_like(params.grad, float("nan"))
    ppo.ppo_loss_grad(ctx, params, batch, dev(np.arange(M, dtype=np.int32), d), ppo.UpdateHParams(), stats, grad, ws)
    torch.cuda.synchronize()
    return grad.cpu().numpy().astype(np.float64)


# splits of two slabs; a shorter last split; a ragged last slab; odd slab
# counts; two splits of a larger network
CASES = [(235, 12, (1024, 512, 256), 512), (235, 12, (1024, 512, 256), 704), (101, 5, (1024, 512, 256), 1000),
         (48, 16, (1024, 512, 256), 4104), (64, 8, (1024, 1024, 512), 256)]


@pytest.mark.parametrize("D,A,H,M", CASES)
def test_paired_tiles(D, A, H, M, monkeypatch, tmp_path):
    d = require_gpu()
    print(f"[gpu-case] paired dw D={D} A={A} H={H} M={M}", flush=True)
    cfg = synth.configs.PPOConfig(name=f"dw_{D}_{A}_{M}", n_envs=8, n_steps=8, net=synth.NetShape(D, A, tuple(H)),
                                  epochs=1, minibatches=1)
    theta = synth.xavier_theta(cfg.net, seed=4, logstd=-0.2)
    batch = {k: dev(v, d) for k, v in teacher_batch(cfg, theta, M, seed=6).items()}
    got = gradient(D, A, H, theta, batch, M, 0, d, monkeypatch, tmp_path)
    ref = gradient(D, A, H, theta, batch, M, 1, d, monkeypatch, tmp_path)
    assert np.isfinite(got).all()
    tol = 2 * 8 * 2.0 ** -24 * np.sqrt(M)
    layout = param_layout(NetSpec(D, A, tuple(H)))
    for name, (off, shape) in layout.items():
        which, _, l = name.partition(".W")
        if not l:
            continue
        n = int(np.prod(shape)) + shape[0]   # the weight, then its bias
        g, r = got[off:off + n], ref[off:off + n]
        worst = np.abs(g - r).max() / (np.sqrt(np.mean(r ** 2)) + 1e-30)
        assert worst <= tol, f"{which} layer {l}: {worst:.3g} of the rms, bound {tol:.3g}"
