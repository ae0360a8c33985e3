"""GAE at the edges of its block rules: one wave per block up to 2^16
environments, four environments per lane from 2^17 on where N is a multiple of
4, one otherwise; horizons around the 8, 16 and 32 steps that load together.
Against the oracle; the statistics against float64 NumPy on the kernel's own
float32 advantages."""
import numpy as np
import pytest
import torch

import paper_2109_11978_amd as ppo
from oracle import gae
from tests.gpu_common import dev, require_gpu
from tests.parity import TOL, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,N", [(1, 2), (31, 63), (32, 64), (33, 65), (65, 130), (3, 1 << 16), (17, (1 << 16) + 1),
                                 (16, (1 << 17) - 1), (8, 1 << 17), (9, (1 << 17) + 4), (7, (1 << 17) + 1028),
                                 (5, (1 << 17) + 3)])
@pytest.mark.parametrize("timeouts", [False, True])
def test_gae_blocks(T, N, timeouts):
    d = require_gpu()
    print(f"[gpu-case] gae T={T} N={N} timeouts={timeouts}", flush=True)
    rng = np.random.default_rng(T * 7 + N)
    r = rng.normal(0, 0.1, (T, N)).astype(np.float32)
    v = rng.normal(3, 1, (T, N)).astype(np.float32)   # a mean that dominates the spread of the errors
    dn = (rng.random((T, N)) < 0.05).astype(np.uint8)
    to = (dn.astype(bool) & (rng.random((T, N)) < 0.5)).astype(np.uint8) if timeouts else None
    last = rng.normal(3, 1, N).astype(np.float32)
    ctx = ppo.Context(8, 2, (16,), "fp32")
    ws = ctx.new_workspace(N=N, T=T)
    out = {}
    for normalize in (False, True):
        adv, ret = torch.empty(T, N, device=d), torch.empty(T, N, device=d)
        st = torch.empty(2, dtype=torch.float64, device=d)
        ppo.ppo_gae(ctx, dev(r, d), dev(dn, d), dev(v, d), dev(last, d), 0.99, 0.95, adv, ret, st,
                    timeouts=dev(to, d) if timeouts else None, normalize=normalize, ws=ws)
        torch.cuda.synchronize()
        out[normalize] = (adv.cpu().numpy(), ret.cpu().numpy(), st.cpu().numpy())
    raw, ret, st = out[False]
    a_ref, r_ref = gae(r, v, dn, last, 0.99, 0.95, timeouts=to)
    assert_close("adv", raw, a_ref, TOL["fp32"])
    assert_close("returns", ret, r_ref, TOL["fp32"])
    x = raw.astype(np.float64)
    mean, std = x.mean(), x.std(ddof=1)
    # float64 sums of T N terms in another order than NumPy's pairwise one
    assert abs(st[0] - mean) <= 1e-12 * np.abs(x).mean() and abs(st[1] - std) <= 1e-12 * std
    assert np.array_equal(out[True][2], st)
    assert np.max(np.abs(out[True][0] - ((x - mean) / (std + 1e-8)))) <= 4 * 2.0 ** -24 * np.max(np.abs(x - mean) / std)


def test_workspace_of_more_environments_serves_fewer():
    ctx = ppo.Context(8, 2, (16,), "fp32")
    sizes = [ctx.workspace_size(N=n, T=8) for n in (1, 64, 4096, (1 << 16) - 1, 1 << 16, (1 << 16) + 1, 1 << 17,
                                                    (1 << 17) + 3, 1 << 20)]
    assert sizes == sorted(sizes)
