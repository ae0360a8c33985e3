"""Plan of the weight-gradient launch (host only): splits by rule."""
import ctypes
import random

import pytest

import paper_2109_11978_amd as ppo

SMALL, LARGE = (512, 256, 128), (1024, 512, 256)


@pytest.fixture(autouse=True)
def _env(monkeypatch):
    for k in ("PPO_AUTOTUNE", "PPO_TUNE_CACHE"):
        monkeypatch.delenv(k, raising=False)


# (precision, inputs, actions, hidden widths, rows, splits, tile height): the
# mini-batches of the flat, rough and large workloads, of the eight-run sweep
# and of a small float32 network.  These are the splits that the tuner's timing
# settled on in most processes when it still chose them (16 to 32 each; 14 of
# 20 at 102400 rows, 13 of 16 at 12288 and at 49152 of the flat network).
CHOICES = [("bf16", 48, 12, SMALL, 24576, 17, 128), ("bf16", 235, 12, SMALL, 24576, 13, 128),
           ("bf16", 235, 12, LARGE, 49152, 4, 128), ("bf16", 48, 12, SMALL, 2048, 5, 64),
           ("bf16", 235, 12, SMALL, 6144, 3, 64), ("bf16", 48, 12, SMALL, 12288, 10, 64),
           ("bf16", 48, 12, SMALL, 32768, 17, 128), ("bf16", 235, 12, SMALL, 73728, 13, 128),
           ("bf16", 48, 12, SMALL, 49152, 17, 128), ("bf16", 235, 12, SMALL, 102400, 6, 128),
           ("fp32", 48, 12, SMALL, 24576, 10, 64), ("fp32", 45, 10, (256, 128, 64), 1001, 8, 64)]


@pytest.mark.parametrize("prec,D,A,H,M,splits,height", CHOICES)
def test_splits_by_rule(prec, D, A, H, M, splits, height):
    plan = ppo.Context(D, A, H, prec).weight_grad_plan(M)
    assert plan["splits"] == splits
    assert (128, 64, 128, 64)[plan["tile"]] == height


def test_plans_cover_the_samples():
    """Every split has samples, in whole k-slabs; the rule's choice is one of
    the tile and round candidates; and the same in every context."""
    rng = random.Random(0)
    for _ in range(300):
        prec = rng.choice(["bf16", "fp32"])
        H = tuple(16 * rng.randint(1, 96) for _ in range(rng.randint(1, 4)))
        D, A, M = rng.randint(1, 500), rng.randint(1, 16), int(2 ** rng.uniform(0, 18))
        ctx = ppo.Context(D, A, H, prec)
        plan = ctx.weight_grad_plan(M)
        assert plan == ppo.Context(D, A, H, prec).weight_grad_plan(M)
        assert plan == ctx.weight_grad_plan(M, plan["tile"], plan["rounds"])
        for tile in range(4):
            for rounds in (1, 2, 4):
                p = ctx.weight_grad_plan(M, tile, rounds)
                s, k = p["splits"], p["samples_per_split"]
                assert (s - 1) * k < M <= s * k and k % (64 if prec == "bf16" else 32) == 0
                assert p["workgroups"] % s == 0


@pytest.mark.parametrize("D,H,M", [(48, (64, 64), 24576), (235, (128, 128), 49152), (300, (128, 128), 98304),
                                   (235, (64, 64), 4096), (235, (512, 256, 128), 1024), (48, (512, 384, 256), 8192),
                                   (235, (1024, 512, 128), 8192)])
def test_narrow_layers_never_pair(D, H, M):
    """A layer of fewer than 256 outputs leaves paired tiles mostly empty."""
    ctx = ppo.Context(D, 12, H, "bf16")
    for rounds in (1, 2, 4):
        assert not ctx.weight_grad_plan(M, 0, rounds)["paired"]
    assert not ctx.weight_grad_plan(M)["paired"]


@pytest.mark.parametrize("D,H,M,splits", [(235, (1024, 512, 256), 49152, 4), (235, (1024, 512, 256), 1000, 4),
                                          (129, (1024, 512, 256), 4104, 4), (256, (1024, 512, 256), 8192, 4),
                                          (48, (512, 512, 256), 24576, 8), (300, (1024, 1024, 512), 98304, 2)])
def test_wide_layers_pair(D, H, M, splits):
    plan = ppo.Context(D, 12, H, "bf16").weight_grad_plan(M, 0, 2)
    assert plan["paired"] and plan["splits"] == splits and 224 <= plan["workgroups"] <= 256
    assert not ppo.Context(D, 12, H, "fp32").weight_grad_plan(M, 0, 2)["paired"]
    assert not ppo.Context(D, 12, H, "bf16").weight_grad_plan(M + 1, 0, 2)["paired"]   # off the buffer-load path


def test_bad_arguments():
    lib, ctx = ppo.load(), ppo.Context(48, 12, (64, 64), "bf16")
    arr = (ctypes.c_int32 * 6)()
    assert lib.ppo_weight_grad_plan(None, 64, -1, 2, arr, 6) == ppo.PPO_E_INVAL
    assert lib.ppo_weight_grad_plan(ctx.handle, 64, -1, 2, None, 6) == ppo.PPO_E_INVAL
    assert lib.ppo_weight_grad_plan(ctx.handle, 64, -1, 2, arr, 5) == ppo.PPO_E_SHAPE
    assert lib.ppo_weight_grad_plan(ctx.handle, 0, -1, 2, arr, 6) == ppo.PPO_E_SHAPE
    assert lib.ppo_weight_grad_plan(ctx.handle, 64, 4, 2, arr, 6) == ppo.PPO_E_INVAL
    assert lib.ppo_weight_grad_plan(ctx.handle, 64, -2, 2, arr, 6) == ppo.PPO_E_INVAL
    assert lib.ppo_weight_grad_plan(ctx.handle, 64, 0, 3, arr, 6) == ppo.PPO_E_INVAL
