"""Column view of many chunks of few entries, whose place blocks share a CU: both sides of the rule (more
chunks of 128 rows than CUs; a mean chunk that fits half a CU's LDS, 9692 entries at 120 columns, 4
at 2888), chunks of more and of fewer than the 4 windows of such a block, and the scan of at most 512
columns, shared by 1024 / n threads from 9 segments of 64 chunks on.  Equal to the stable sort by
column, exactly."""
import numpy as np
import pytest
import torch

from paper_2508_07605_amd import native

pytestmark = pytest.mark.gpu
CUS = 256


@pytest.mark.parametrize("m,n,hi,full", [
    (128 * CUS, 120, 3, 0), (128 * CUS + 1, 120, 3, 0), (128 * CUS + 1, 120, 3, 128),
    (128 * (CUS + 9), 120, 120, 0), (128 * (CUS + 9), 76, 76, 128 * (CUS + 9)),
    (128 * (CUS + 9), 77, 77, 128 * (CUS + 9)), (128 * (CUS + 9), 284, 2, 200), (128 * (CUS + 9), 285, 2, 200),
    (128 * (CUS + 9), 1920, 2, 30),
    (128 * (CUS + 9), 2888, 0, 1), (128 * (CUS + 9), 2889, 1, 5),
    (65536, 480, 2, 0), (65537, 480, 2, 0), (65537, 512, 2, 0),
    (300001, 1, 1, 0), (300001, 2, 2, 0), (300001, 3, 3, 0), (100003, 511, 2, 3), (100003, 512, 2, 3),
    (100003, 513, 2, 3), (63, 512, 5, 1), (1, 1, 1, 1), (1100003, 7, 2, 300)])
def test_sparse_chunks(m, n, hi, full):
    r = np.random.default_rng([m, n, hi, full])
    counts = r.integers(0, hi + 1, size=m)
    start = m // 3 if full < m else 0
    counts[start:start + full] = n
    rp = np.zeros(m + 1, np.int64)
    rp[1:] = np.cumsum(counts)
    rows = np.repeat(np.arange(m), counts)
    col = ((np.arange(len(rows)) - rp[rows] + r.integers(0, n, size=m)[rows]) % n).astype(np.int32)
    val = r.uniform(size=len(col)).astype(np.float32)
    dev = lambda a: torch.from_numpy(a).cuda()
    ctx = native.Context(0)
    try:
        cp, ri, cv = native.open_csr_to_csc(ctx, dev(rp), dev(col), dev(val), n)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    order = np.argsort(col, kind="stable")
    assert np.array_equal(cp.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(col, minlength=n))]))
    assert np.array_equal(ri.cpu().numpy(), rows[order])
    assert np.array_equal(cv.cpu().numpy(), val[order])
