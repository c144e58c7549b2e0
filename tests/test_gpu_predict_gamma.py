"""Algorithm 2 at loss bounds near 1, where the float32 rounding of 1 - p / p_base spans many units
in the last place of p: every row's settings lie around the least prediction that the rule
accepts, in steps down to one unit, and are priced so that the lowest accepted one is the pick.
The pick, saving and status are those of the rule applied in float32 to the kernel's own
prediction, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2508_07605_amd import native

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gamma", [0.0, 0.05, 0.9, 0.995, 0.999, 0.9999, 0.99999, 0.999999, 1.0 - 2.0 ** -24])
@pytest.mark.parametrize("k", [8, 64])
def test_least_accepted_prediction(k, gamma):
    gamma = np.float32(gamma)
    r = np.random.default_rng([k, int(1e7 * float(gamma))])
    one = np.float32(1)
    m, n = 160, 420
    U = np.zeros((m, k), np.float32)
    U[:, 1] = np.concatenate([np.exp(r.uniform(-3, 3, m - 4)), [1.0, 1e-30, 1e30, 1e-38]])
    v0 = one - gamma
    # the accepted set of a row with p_base = 1 starts within v0 - 2^-24 .. v0 + 2^-24
    steps = np.arange(-100, 101, dtype=np.int64)
    near = np.maximum(np.array(v0, np.float32).view(np.int32) + steps, 1).astype(np.int32).view(np.float32)
    wide = v0 + np.float32(2.0 ** -24) * np.linspace(-1.5, 1.5, n - 1 - len(near)).astype(np.float32)
    V = np.zeros((n, k), np.float32)
    V[:, 1] = np.concatenate([near, np.maximum(wide, 2.0 ** -26), [1.0]])
    base = n - 1
    # cost ~ v^2: the key p / cost falls as p grows
    c = (1e3 * V[:, 1].astype(np.float64) ** 2).astype(np.float32)
    g = c.copy()
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    ctx = native.Context(0)
    try:
        P = torch.empty((m, n), device="cuda")
        st = torch.empty(m, dtype=torch.int32, device="cuda")
        d = [dev(x) for x in (U, V, c, g)]
        idx, sav = native.open_predict(ctx, *d, base, float(gamma), P=P, row_status=st)
        idx2, _ = native.open_predict(ctx, *d, base, float(gamma))
        idx, sav, st, p = idx.cpu().numpy(), sav.cpu().numpy(), st.cpu().numpy(), P.cpu().numpy()
        assert np.array_equal(idx, idx2.cpu().numpy())
    finally:
        ctx.close()
    cost = c + g
    with np.errstate(all="ignore"):
        pb = p[:, base:]
        ok = (p > 0) & (pb > 0) & ((one - p / pb) <= gamma)
        key = np.where(ok, p * (one / cost), -np.inf)
        pick = np.argmax(key, axis=1)
        good = ok.any(axis=1)
        E = cost[pick] / p[np.arange(m), pick]
        want = np.where(good, (cost[base] - E) / cost[base], np.float32(0))
    assert ok[:, :base].any() and not ok[:, :base].all()
    np.testing.assert_array_equal(idx, np.where(good, pick, base))
    np.testing.assert_array_equal(sav, want.astype(np.float32))
    np.testing.assert_array_equal(st == 0, good)
