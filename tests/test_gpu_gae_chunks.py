"""GAE at every kernel of its rule and around the rule's edges, against the
oracle; the statistics against float64 NumPy on the kernel's own advantages."""
import numpy as np
import pytest
import torch

import paper_2109_11978_amd as ppo
from oracle import gae
from tests.gpu_common import dev, require_gpu
from tests.parity import TOL, assert_close

pytestmark = pytest.mark.gpu

SMALL = [(T, N) for T in (7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 47, 48, 49, 64, 65, 100) for N in (65, 4096)]
# edges of the rule: 49152, 65536, 131072, 163840 and 262144 environments; 24, 64, 96 and 256 steps
MEDIUM = [(T, N) for T in (24, 25, 256, 257) for N in (49152, 49153, 65536, 65537)]
LARGE = [(T, N) for T in (1, 7, 9, 96, 97) for N in (131072, 131076, 131073, 163836, 163840)]
MANY = [(T, N) for T in (1, 4, 5, 64, 65) for N in (262140, 262144, 263172, 262145)]


@pytest.mark.parametrize("T,N", SMALL + MEDIUM + LARGE + MANY)
def test_gae_chunks(T, N):
    d = require_gpu()
    print(f"[gpu-case] gae chunks T={T} N={N}", flush=True)
    rng = np.random.default_rng(T * 7 + N)
    r = rng.normal(0, 0.1, (T, N)).astype(np.float32)
    v = rng.normal(3, 1, (T, N)).astype(np.float32)
    dn = (rng.random((T, N)) < 0.05).astype(np.uint8)
    to = (dn.astype(bool) & (rng.random((T, N)) < 0.5)).astype(np.uint8)
    last = rng.normal(3, 1, N).astype(np.float32)
    ctx = ppo.Context(8, 2, (16,), "fp32")
    adv, ret = torch.empty(T, N, device=d), torch.empty(T, N, device=d)
    st = torch.empty(2, dtype=torch.float64, device=d)
    ppo.ppo_gae(ctx, dev(r, d), dev(dn, d), dev(v, d), dev(last, d), 0.99, 0.95, adv, ret, st, timeouts=dev(to, d),
                normalize=False, ws=ctx.new_workspace(N=N, T=T))
    torch.cuda.synchronize()
    a_ref, r_ref = gae(r, v, dn, last, 0.99, 0.95, timeouts=to)
    raw = adv.cpu().numpy()
    assert_close("adv", raw, a_ref, TOL["fp32"])
    assert_close("returns", ret.cpu().numpy(), r_ref, TOL["fp32"])
    x = raw.astype(np.float64)
    mean, std = x.mean(), x.std(ddof=1)
    st = st.cpu().numpy()
    # float64 sums of T N terms in another order than NumPy's pairwise one
    assert abs(st[0] - mean) <= 1e-12 * np.abs(x).mean() and abs(st[1] - std) <= 1e-12 * std
