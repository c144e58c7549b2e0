"""The fused prediction and selection at the edges of its tiles (32 rows by 32 settings): the pick,
the saving and the status follow, bit for bit, from the paper's rule applied in float32 to the
prediction that the kernel itself writes, with and without that prediction asked for, with equal
settings (the lowest wins), rows without a valid baseline, NaN rows and every loss bound."""
import numpy as np
import pytest
import torch

from paper_2508_07605_amd import native

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gamma", [0.0, 0.05, 1.5])
@pytest.mark.parametrize("k,m,n", [(8, 1, 1), (8, 257, 33), (16, 31, 65), (16, 130, 32), (32, 33, 31), (32, 129, 96),
                                   (64, 127, 97), (64, 160, 64)])
def test_rule_on_own_prediction(k, m, n, gamma):
    ctx = native.Context(0)
    r = np.random.default_rng(m + n)
    U = r.uniform(0.0, 1.0, (m, k)).astype(np.float32)
    V = r.uniform(0.2, 1.0, (n, k)).astype(np.float32)
    c, g = r.uniform(50, 400, n).astype(np.float32), r.uniform(100, 700, n).astype(np.float32)
    if n > 2:  # equal settings: equal keys
        for a, b in ((0, n - 1), (1, n // 2)):
            V[b], c[b], g[b] = V[a], c[a], g[a]
    U[m // 2] = -U[m // 2]  # p_base < 0
    if m > 3:
        U[3] = np.nan
    base = n - 1
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    d = [dev(x) for x in (U, V, c, g)]
    outs = []
    for want in (True, False):
        P = torch.empty((m, n), device="cuda") if want else None
        st = torch.empty(m, dtype=torch.int32, device="cuda")
        idx, sav = native.open_predict(ctx, *d, base, gamma, P=P, row_status=st)
        outs.append((idx.cpu().numpy(), sav.cpu().numpy(), st.cpu().numpy()))
        if want:
            p = P.cpu().numpy()
    for a, b in zip(*outs):
        np.testing.assert_array_equal(a, b)
    one = np.float32(1)
    cost = c + g
    with np.errstate(all="ignore"):
        pb = p[:, base:base + 1]
        ok = (p > 0) & (pb > 0) & ((one - p / pb) <= np.float32(gamma))
        key = np.where(ok, p * (one / cost), -np.inf)
        pick = np.argmax(key, axis=1)
        good = ok.any(axis=1)
        E = cost[pick] / p[np.arange(m), pick]
        sav = np.where(good, (cost[base] - E) / cost[base], np.float32(0))
    idx, got, st = outs[0]
    np.testing.assert_array_equal(idx, np.where(good, pick, base))
    np.testing.assert_array_equal(got, sav.astype(np.float32))
    np.testing.assert_array_equal(st == 0, good)
    ctx.close()
