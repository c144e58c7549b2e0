"""The NCF fold-in with four applications per wavefront (large batches) against the one with two:
the same applications in batches small enough for the latter give the same bits, whatever their
neighbours, for every way that their observations can fill the tiles (none, one shared, full
ones, both), ragged batches and every status."""
import numpy as np
import pytest
import torch

from paper_2508_07605_amd import native, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lo,hi,extra", [(1, 8, 1), (7, 18, 2), (9, 16, 3), (15, 26, 4), (24, 42, 5)])
def test_two_pairs_match_one(lo, hi, extra):
    ctx = native.Context(0)
    n, steps = 120, 3
    m = 24 * torch.cuda.get_device_properties(0).multi_processor_count + extra  # just past the rule
    r = np.random.default_rng(lo)
    counts = r.integers(lo, hi + 1, size=m)
    counts[[0, m // 2, m - 1]] = 0
    rp = np.zeros(m + 1, np.int64)
    rp[1:] = np.cumsum(counts)
    col = r.integers(0, n, size=int(rp[-1])).astype(np.int32)
    val = r.uniform(0.4, 1.0, size=int(rp[-1])).astype(np.float32)
    col[rp[5]] = n            # refused: setting out of range
    val[rp[m - 6]] = np.inf   # refused: not finite
    p = synth.ncf_params(3, n, seed=lo)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    S = dev(p.pop("S"))
    net = {k: dev(v) for k, v in p.items()}

    def fold(a, b):
        sl = slice(int(rp[a]), int(rp[b]))
        loss, st = torch.empty(b - a, device="cuda"), torch.empty(b - a, dtype=torch.int32, device="cuda")
        E = native.open_ncf_foldin(ctx, S, net, dev(rp[a:b + 1] - rp[a]), dev(col[sl]), dev(val[sl]), steps, 0.5, 1e-3,
                                   loss_out=loss, row_status=st)
        return E.cpu(), loss.cpu(), st.cpu()

    whole = fold(0, m)
    cuts = [0, m // 3 - 1, 2 * (m // 3) + 2, m]
    parts = [fold(a, b) for a, b in zip(cuts[:-1], cuts[1:])]
    for w, q in zip(whole, zip(*parts)):
        assert torch.equal(w, torch.cat(q))
    st = whole[2].numpy()
    assert st[0] == 1 and st[5] == 5 and st[m - 6] == 3 and np.isfinite(whole[0].numpy()).all()
    ctx.close()
