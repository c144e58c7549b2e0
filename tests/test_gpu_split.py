"""Split-K rows whose parts follow the XCDs' ranges of a factor matrix larger than an L2, and the
plain parts beside it, at every rank: rows of just the split length, of no multiple of eight or of
an accumulator's 1024 entries, and one that fills the matrix; with too many rows for ranges.
Per-row relative error against the float64 oracle at most 1e-4, the bound of the other ridge
tests; statuses equal."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_07605_amd import native

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = native.Context(0)
    yield c
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("k", [8, 16, 32, 64])
@pytest.mark.parametrize("n,short", [(70_001, 20), (70_001, 4100), (1500, 20)])
def test_long_rows(ctx, k, n, short):
    # 70,001 rows of factors exceed 2 MB at every rank; 4100 further rows put the matrix past
    # the row count up to which parts follow ranges
    r = np.random.default_rng([k, n, short])
    longs = [1024, 1025, 1031, min(n, 8191), min(n, 12_345), n]
    counts = np.concatenate([longs, r.integers(0, 20, size=short)])
    r.shuffle(counts)
    rp = np.zeros(len(counts) + 1, np.int64)
    rp[1:] = np.cumsum(counts)
    col = np.concatenate([np.sort(r.choice(n, size=c, replace=False)) for c in counts]).astype(np.int32)
    val = r.uniform(0.4, 1.0, size=len(col)).astype(np.float32)
    F = (0.3 * r.normal(size=(n, k))).astype(np.float32)
    bad = np.nonzero(counts == 12_345)[0]
    if len(bad):
        val[rp[bad[0]] + 9000] = np.nan
    ill = np.nonzero(counts == min(n, 8191))[0][0]
    col[rp[ill] + 1100] = n + 3
    st = torch.full((len(counts),), -7, dtype=torch.int32, device="cuda")
    U = native.open_foldin(ctx, dev(F), dev(rp), dev(col), dev(val), 0.05, True, row_status=st)
    torch.cuda.synchronize()
    U, st = U.cpu().numpy().astype(np.float64), st.cpu().numpy()
    assert st[ill] == 5 and (U[ill] == 0).all()
    ok = np.ones(len(counts), bool)
    ok[ill] = False
    if len(bad):
        assert st[bad[0]] == 3 and (U[bad[0]] == 0).all()
        ok[bad] = False
    col[rp[ill] + 1100] = 0
    ref, ref_st = oracle.ridge_rows(rp, col, np.nan_to_num(val), F, 0.05, True)
    assert np.array_equal(st[ok], ref_st[ok])
    nrm = np.linalg.norm(ref, axis=1)
    e = np.linalg.norm(U - ref, axis=1) / np.where(nrm > 0, nrm, 1.0)
    print("k %d n %d: %d rows, max error %.2e" % (k, n, len(counts), e[ok].max()))
    assert e[ok].max() <= 1e-4
    # the same again: the result does not depend on scheduling
    U2 = native.open_foldin(ctx, dev(F), dev(rp), dev(np.where(np.arange(len(col)) == rp[ill] + 1100, n + 3, col)),
                            dev(val), 0.05, True)
    assert np.array_equal(U2.cpu().numpy()[ok], U[ok].astype(np.float32))
