"""Split-K parts of many thousand entries: the right-hand side, like the Gram matrix, is summed in
pieces of 1024 entries, so its error does not grow with the part.  And rows of many parts.

Every row observes all 262,144 factor rows, whose columns are those of a Hadamard matrix (entries
+-1, exactly orthogonal): the Gram matrix is 262,144 I without rounding, and the solution is the
right-hand side over 262,144 + lambda.  With the row counts below a row has eight parts of 32,768
entries, 8192 terms a lane.  The value observed, the same everywhere, is 0.499 units of 2^-11 above
a multiple of 2^-11, so a running sum between 4096 and 8192 is rounded down at every term: one chain
over a part would be off by 1e-4.

Tolerance: the first unknown is the only one that is not zero.  Its right-hand side is summed from
256 terms (half a unit in the last place, 2^-24 of the sum, each at most), 32 such pieces, 4 lanes
and 8 parts, the others' from as many terms of the same size; the rest of the solve is 8 roundings."""
import numpy as np
import pytest
import torch

from paper_2508_07605_amd import native

pytestmark = pytest.mark.gpu

N = 262_144
VALUE = np.float32((1433 + 0.499) * 2.0 ** -11)


@pytest.mark.parametrize("k,m", [(8, 512), (16, 512), (32, 512), (64, 256)])
def test_right_hand_side_of_long_parts(k, m):
    j, d = np.arange(N)[:, None], np.arange(k)[None, :]
    x = j & d
    for s in (8, 4, 2, 1):
        x ^= x >> s
    F = torch.from_numpy(np.where(x & 1, -1.0, 1.0).astype(np.float32)).cuda()
    rp = torch.arange(m + 1, dtype=torch.int64, device="cuda") * N
    col = torch.arange(N, dtype=torch.int32, device="cuda").repeat(m)
    val = torch.full((m * N,), float(VALUE), device="cuda")
    lam = 0.5
    ctx = native.Context(0)
    try:
        U = native.open_foldin(ctx, F, rp, col, val, lam, False)
        torch.cuda.synchronize()
        U = U.cpu().numpy().astype(np.float64)
    finally:
        ctx.close()
    want = np.zeros(k)
    want[0] = float(VALUE) * N / (N + lam)
    rel = np.abs(U - want).max(axis=1) / want[0]
    print("k %d: max error %.2e of the solution" % (k, rel.max()))
    assert rel.max() <= (256 + 32 + 4 + 8 + 8) * 2.0 ** -24


@pytest.mark.parametrize("k", [8, 16, 32, 64])
@pytest.mark.parametrize("counts", [[100_000], [1024, 149_999, 30_000], [150_000] * 5 + [9_000]])
def test_rows_of_many_parts(k, counts):
    """Few rows of very different lengths, cut into many parts each: per-row relative error against
    float64 at most 1e-4, the bound of the other ridge tests, and the same bits again."""
    n = 150_000
    r = np.random.default_rng([k, len(counts)])
    rp = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    col = np.concatenate([np.sort(r.choice(n, size=c, replace=False)) for c in counts]).astype(np.int32)
    val = r.uniform(0.4, 1.0, size=len(col)).astype(np.float32)
    F = (0.3 * r.normal(size=(n, k))).astype(np.float32)
    dev = [torch.from_numpy(a).cuda() for a in (F, rp, col, val)]
    ctx = native.Context(0)
    try:
        st = torch.full((len(counts),), -7, dtype=torch.int32, device="cuda")
        U = native.open_foldin(ctx, *dev, 0.05, True, row_status=st).cpu().numpy()
        again = native.open_foldin(ctx, *dev, 0.05, True).cpu().numpy()
        assert (st == 0).all()
    finally:
        ctx.close()
    assert np.array_equal(U, again)
    for i, c in enumerate(counts):
        A, b = F[col[rp[i]:rp[i + 1]]].astype(np.float64), val[rp[i]:rp[i + 1]].astype(np.float64)
        ref = np.linalg.solve(A.T @ A + 0.05 * c * np.eye(k), A.T @ b)
        assert np.linalg.norm(U[i] - ref) <= 1e-4 * np.linalg.norm(ref)
