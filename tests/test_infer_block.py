"""The block that inference runs in (host only)."""
import ctypes

import pytest

import paper_2109_11978_amd as ppo


@pytest.fixture(autouse=True)
def _env(monkeypatch):
    for k in ("PPO_FUSED", "PPO_FUSED_ROWS", "PPO_FUSED_THREADS", "PPO_FUSED_PER_CU"):
        monkeypatch.delenv(k, raising=False)


@pytest.mark.parametrize("D,A,H,prec,block", [
    (48, 12, (512, 256, 128), "bf16", (32, 256)),      # the general block
    (235, 12, (512, 256, 128), "bf16", (32, 256)),     # 235 inputs pad to 240
    (225, 12, (512, 256, 128), "bf16", (32, 256)),     # 225 to 232, no multiple of 16
    (48, 12, (64, 64), "bf16", (32, 128)),             # narrow
    (235, 12, (1024, 512, 256), "bf16", (64, 512)),    # wide
    (235, 12, (2048, 512, 256), "bf16", (0, 0)),       # wider than the wide pass holds
    (48, 3, (512, 256, 128), "bf16", (0, 0)),          # misaligned critic biases
    (48, 12, (512, 256, 128), "fp32", (0, 0)),
])
def test_infer_block(D, A, H, prec, block, monkeypatch):
    ctx = ppo.Context(D, A, H, prec)
    assert ctx.infer_block() == block
    if ctx.fused_infer_shape() != (0, 0) and A == 12:
        assert ctx.fused_infer_shape() == block
    monkeypatch.setenv("PPO_FUSED", "0")
    assert ctx.infer_block() == (0, 0)


def test_forced_shape(monkeypatch):
    monkeypatch.setenv("PPO_FUSED_ROWS", "64")
    monkeypatch.setenv("PPO_FUSED_THREADS", "512")
    assert ppo.Context(48, 12, (512, 256, 128), "bf16").infer_block() == (64, 512)
    assert ppo.Context(48, 12, (64, 64), "bf16").infer_block() == (0, 0)


def test_bad_arguments():
    lib, ctx, v = ppo.load(), ppo.Context(48, 12, (64, 64), "bf16"), ctypes.c_int32()
    assert lib.ppo_infer_block(None, ctypes.byref(v), ctypes.byref(v)) == ppo.PPO_E_INVAL
    assert lib.ppo_infer_block(ctx.handle, None, ctypes.byref(v)) == ppo.PPO_E_INVAL
    assert lib.ppo_infer_block(ctx.handle, ctypes.byref(v), None) == ppo.PPO_E_INVAL
