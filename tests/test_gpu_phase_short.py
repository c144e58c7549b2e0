"""Algorithm 1 on more short traces than wavefronts (each then takes several) and at the lengths where
the number of steps loaded together changes: exact against the rule in numpy."""
import numpy as np
import pytest
import torch

from paper_2508_07605_amd import native

pytestmark = pytest.mark.gpu


def detect(P, th, n):
    """First position whose run of readings not below th reaches n, per trace; -1 without one."""
    ok = ~(P < th)
    idx = np.arange(P.shape[1])
    last = np.maximum.accumulate(np.where(ok, -1, idx), axis=1)  # last failing reading so far
    hit = (idx - last >= n) & ok
    return np.where(hit.any(axis=1), hit.argmax(axis=1), -1)


@pytest.mark.parametrize("L", [1, 2, 40, 63, 64, 65, 127, 128, 129, 256, 300, 768, 769])
def test_many_short_traces(L):
    r = np.random.default_rng(L)
    T = 64 * 256 * 2 + 77  # two rounds and a remainder on a card of 256 units
    keep = r.choice(np.array([0.5, 0.9, 0.97, 0.99, 1.0]), size=(T, 1))
    P = np.where(r.random((T, L)) < keep, np.float32(100), np.float32(10)).astype(np.float32)
    P[::7] = 10.0
    P[3::11, : L // 2] = 10.0
    P[5::13, L - 1] = np.nan
    P[6::17, 0] = 60.0
    d = torch.from_numpy(P).cuda()
    ctx = native.Context(0)
    try:
        for n in (1, 2, 25, 64, 65, 130):
            got = native.open_phase_detect(ctx, d, 60.0, n)
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), detect(P, np.float32(60), n)), n
    finally:
        ctx.close()
