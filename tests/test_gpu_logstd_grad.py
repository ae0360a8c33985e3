"""Log-std gradient of single samples whose actions lie one standard deviation
from the mean, where z^2 - 1 cancels.  With every weight zero the means and
log-stds are exactly zero, so z is the action, and with one sample the
gradient is -adv ratio (z_j^2 - 1): relative to the dimension with z = 2 it is
(z_j^2 - 1) / 3.  The subtraction is one rounding of the exact z^2 - 1, so the
quotient is within 4 float32 roundings of the exact one; a z^2 rounded by
itself would be up to 2^-13 off at these z."""
import numpy as np
import pytest
import torch

import paper_2109_11978_amd as ppo
from tests.gpu_common import dev, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("D,A,H,prec", [(48, 12, (512, 256, 128), "bf16"), (235, 16, (512, 256, 128), "bf16"),
                                        (48, 5, (256, 128, 64), "bf16"), (45, 7, (64, 64), "bf16"),
                                        (48, 12, (1024, 512, 256), "bf16"), (45, 7, (64, 64), "fp32")])
def test_one_sample(D, A, H, prec, fused, monkeypatch):
    d = require_gpu()
    monkeypatch.setenv("PPO_FUSED", "1" if fused else "0")
    monkeypatch.setenv("PPO_AUTOTUNE", "0")
    print(f"[gpu-case] logstd D={D} A={A} H={H} {prec} fused={fused}", flush=True)
    ctx = ppo.Context(D, A, H, prec)
    p = ppo.Params(ctx, np.zeros(ctx.param_count, np.float32), device=d)
    # odd multiples of 2^-12 above or below one: z^2 needs one bit more than float32 has
    z = (1.0 + np.arange(-2 * A + 1, 2 * A, 4) * 2.0 ** -12).astype(np.float32)[:A]
    z[0] = 2.0
    logp = -0.5 * np.sum(z.astype(np.float64) ** 2) - 0.5 * A * np.log(2 * np.pi)
    batch = dict(obs=np.zeros((1, D), np.float32), actions=z[None], logp=np.float32([logp]), adv=np.float32([1]),
                 returns=np.float32([0]))
    grad, stats = torch.empty_like(p.grad), torch.zeros(ppo.PPO_STATS_WIDTH, device=d)
    ppo.ppo_loss_grad(ctx, p, {k: dev(v, d) for k, v in batch.items()}, dev(np.zeros(1, np.int32), d),
                      ppo.UpdateHParams(entropy_coef=0.0), stats, grad, ctx.new_workspace(M=1))
    torch.cuda.synchronize()
    at = ctx.param_offsets()[2 * (len(H) + 1)]
    g = grad.cpu().numpy().astype(np.float64)[at:at + A]
    exact = (z.astype(np.float64) ** 2 - 1) / 3
    assert g[0] != 0
    assert np.max(np.abs(g / g[0] / exact - 1)) <= 4 * 2.0 ** -24
