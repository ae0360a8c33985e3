"""The tile query after one-launch inference of many row counts: it answers for
the latest of them, keeps a bounded number and refuses counts that never ran."""
import pytest
import torch

import paper_2109_11978_amd as ppo
import synth
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


def test_many_row_counts():
    d = require_gpu()
    net = synth.NetShape(48, 12, (64, 64))
    ctx = ppo.Context(48, 12, (64, 64), "bf16")
    params = ppo.Params(ctx, synth.xavier_theta(net, seed=3, logstd=-0.25), device=d)
    obs, ws = torch.zeros(200, 48, device=d), ctx.new_workspace(N=200)
    for n in list(range(1, 150)) + [149, 148, 149]:
        ppo.ppo_rollout_infer(ctx, params, obs[:n], t=0, seed=1, iteration=0, ws=ws, values=torch.empty(n, device=d))
    torch.cuda.synchronize()
    for n in range(149 - 63, 150):
        assert ctx.tuning(n, False)["forward_1"] == "128x128"
    for n in (1, 149 - 64, 150):
        with pytest.raises(ppo.PPOError):
            ctx.tuning(n, False)
