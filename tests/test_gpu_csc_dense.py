"""Column view of chunks of 128 rows with too many entries for their windows in LDS, which are stored
as ranked: both sides of the rule (12 windows, of 10,240 entries, or 5632 at 4096 columns), full
rows, a chunk of either kind in one matrix, and columns in any order within a row.  Equal to the
stable sort by column, exactly."""
import numpy as np
import pytest
import torch

from paper_2508_07605_amd import native

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,lo,hi", [(256, 1920, 960, 960), (256, 1920, 961, 961), (200, 4096, 528, 528),
                                       (200, 4096, 529, 529), (130, 4096, 4096, 4096), (700, 4096, 200, 900),
                                       (259, 2500, 2500, 2500)])
@pytest.mark.parametrize("shuffled", [False, True])
def test_dense_rows(m, n, lo, hi, shuffled):
    r = np.random.default_rng([m, n, lo, int(shuffled)])
    counts = r.integers(lo, hi + 1, size=m)
    rp = np.zeros(m + 1, np.int64)
    rp[1:] = np.cumsum(counts)
    pick = [r.choice(n, size=c, replace=False) for c in counts]
    col = np.concatenate([p if shuffled else np.sort(p) for p in pick]).astype(np.int32)
    val = r.uniform(size=len(col)).astype(np.float32)
    dev = lambda a: torch.from_numpy(a).cuda()
    ctx = native.Context(0)
    try:
        cp, ri, cv = native.open_csr_to_csc(ctx, dev(rp), dev(col), dev(val), n)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    rows = np.repeat(np.arange(m), counts)
    order = np.lexsort((rows, col))
    assert np.array_equal(cp.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(col, minlength=n))]))
    assert np.array_equal(ri.cpu().numpy(), rows[order])
    assert np.array_equal(cv.cpu().numpy(), val[order])
