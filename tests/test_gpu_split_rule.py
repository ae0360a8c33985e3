"""An update's result does not depend on the tuner's timing: contexts that tune
afresh give the same bits, at row counts where the weight gradient's split
counts lie within a few per cent of each other."""
import numpy as np
import pytest
import torch

import paper_2109_11978_amd as ppo
import synth
from tests.gpu_common import dev, require_gpu, teacher_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,A,H,prec,M", [(48, 12, (512, 256, 128), "bf16", 2048),
                                          (235, 12, (512, 256, 128), "bf16", 6144),
                                          (48, 12, (512, 256, 128), "bf16", 12288),
                                          (48, 12, (512, 256, 128), "bf16", 2001),
                                          (235, 12, (1024, 512, 256), "bf16", 4096),
                                          (45, 10, (256, 128, 64), "fp32", 2048)])
def test_fresh_contexts_agree(D, A, H, prec, M, monkeypatch):
    d = require_gpu()
    monkeypatch.delenv("PPO_TUNE_CACHE", raising=False)
    monkeypatch.delenv("PPO_AUTOTUNE", raising=False)
    print(f"[gpu-case] split rule D={D} A={A} H={H} {prec} M={M}", flush=True)
    cfg = synth.configs.PPOConfig(name=f"split_{D}_{A}_{M}", n_envs=8, n_steps=8, net=synth.NetShape(D, A, tuple(H)),
                                  epochs=1, minibatches=1)
    theta = synth.xavier_theta(cfg.net, seed=4, logstd=-0.2)
    small = teacher_batch(cfg, theta, 256, seed=6)
    batch = {k: dev(np.concatenate([v] * (M // 256 + 1))[:M], d) for k, v in small.items()}
    first = None
    for _ in range(10):
        ctx = ppo.Context(D, A, H, prec)
        p = ppo.Params(ctx, theta, device=d)
        grad, stats = torch.empty_like(p.grad), torch.zeros(ppo.PPO_STATS_WIDTH, device=d)
        ppo.ppo_loss_grad(ctx, p, batch, dev(np.arange(M, dtype=np.int32), d), ppo.UpdateHParams(), stats, grad,
                          ctx.new_workspace(M=M))
        first = grad.clone() if first is None else first
        assert torch.equal(grad, first)


@pytest.mark.parametrize("prec", ["bf16", "fp32"])
def test_tiles_of_one_height_agree(prec):
    """What is left to timing keeps the bits: weight-gradient tiles of one
    height and split, sums of rows included."""
    d = require_gpu()
    print(f"[gpu-case] dw tiles {prec}", flush=True)
    M, N, K, splits = 200, 136, 1064, 3
    dt = torch.bfloat16 if prec == "bf16" else torch.float32
    g = torch.Generator(device=d)
    g.manual_seed(3)
    a = torch.randn(K, M, device=d, generator=g).to(dt).contiguous()
    b = torch.randn(K, N, device=d, generator=g).to(dt).contiguous()
    lib = ppo.load()
    out = {}
    for tile in range(4):
        c = torch.full((splits, M, N), float("nan"), device=d)
        rows = torch.full((splits, M), float("nan"), device=d)
        assert lib.ppo_gemm_check(torch.cuda.current_stream().cuda_stream, 1 if prec == "bf16" else 0, 1, 1, 2, M, N, K,
                                  a.data_ptr(), M, b.data_ptr(), N, c.data_ptr(), N, None, None, 0, rows.data_ptr(),
                                  splits, tile) == 0
        torch.cuda.synchronize()
        out[tile] = (c, rows)
    for x, y in ((0, 2), (1, 3)):
        assert torch.equal(out[x][0], out[y][0]) and torch.equal(out[x][1], out[y][1])
    assert torch.equal(out[0][0], out[1][0])   # the products agree over all four
