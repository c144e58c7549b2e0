"""Factor matrices of 4 GiB and more, where 32-bit byte offsets no longer reach every row: rows of
every size class at each rank, with indices on both sides of 4 GiB, rejected ones, and the row that
the offset of index -1 would wrap to filled with large numbers; and the largest matrix still within
reach.  Per-row relative error against float64 at most 1e-4, the bound of the other ridge tests."""
import numpy as np
import pytest
import torch

from paper_2508_07605_amd import native

pytestmark = pytest.mark.gpu

LAM = 0.05


def solve64(A, b, cnt, weighted):
    return np.linalg.solve(A.T @ A + LAM * (cnt if weighted else 1) * np.eye(A.shape[1]), A.T @ b)


@pytest.mark.parametrize("k,more", [(8, 1000), (16, 1000), (32, 1000), (64, 1000), (64, 0), (64, -1)])
@pytest.mark.parametrize("weighted", [True, False])
def test_fold_in(k, more, weighted):
    n = 2 ** 32 // (4 * k) + more
    r = np.random.default_rng([k, more + 1, int(weighted)])
    counts = np.array([3, 4, 7, 12, 15, 19, 22, 26, 31, 32, 33, 40, 64, 65, 100, 300, 1023, 1024, 1025, 5000, 0, 6, 50, 2000])
    wrap = 2 ** 32 // (4 * k) - 1
    cols = []
    for c in counts:
        j = np.concatenate([r.integers(0, 1000, size=c // 3), r.integers(n - 900, n, size=c - c // 3)])
        j = np.where(j == wrap, wrap - 950, j)
        if c > 900:
            j = r.choice(n // 1000, size=c, replace=False).astype(np.int64) * 1000 + 7
        cols.append(np.unique(j))
    counts = np.array([len(j) for j in cols])
    rp = np.zeros(len(counts) + 1, np.int64)
    rp[1:] = np.cumsum(counts)
    col = np.concatenate(cols).astype(np.int32)
    val = r.uniform(0.4, 1.0, size=len(col)).astype(np.float32)
    used, where = np.unique(col, return_inverse=True)
    rows = (0.3 * r.normal(size=(len(used), k))).astype(np.float32)
    F = torch.zeros((n, k), device="cuda")
    if wrap < n:
        F[wrap] = 50.0
    F[torch.from_numpy(used.astype(np.int64)).cuda()] = torch.from_numpy(rows).cuda()
    bad = [len(counts) - 3, len(counts) - 2, len(counts) - 1]  # a short, a primal and a long row
    for i, x in zip(bad, (n, -1, n + 5)):
        col[rp[i] + 2] = x
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ctx = native.Context(0)
    try:
        st = torch.full((len(counts),), -7, dtype=torch.int32, device="cuda")
        U = native.open_foldin(ctx, F, dev(rp), dev(col), dev(val), LAM, weighted, row_status=st)
        torch.cuda.synchronize()
        U, st = U.cpu().numpy().astype(np.float64), st.cpu().numpy()
    finally:
        ctx.close()
    del F
    worst = 0.0
    for i, c in enumerate(counts):
        if i in bad or c == 0:
            assert st[i] == (5 if c else 1) and (U[i] == 0).all()
            continue
        A, b = rows[where[rp[i]:rp[i + 1]]].astype(np.float64), val[rp[i]:rp[i + 1]].astype(np.float64)
        ref = solve64(A, b, c, weighted)
        e = np.linalg.norm(U[i] - ref) / np.linalg.norm(ref)
        assert st[i] == 0 and e <= 1e-4, (k, n, c, e)
        worst = max(worst, e)
    print("k %d, %d rows of factors: max error %.2e" % (k, n, worst))


def test_fit_columns():
    """Column half-sweep over more than 4 GiB of application factors: V solves its normal equations for
    the U returned, to 1e-4 of the right-hand side."""
    k, n, m = 64, 12, 2 ** 24 + 5000
    g = torch.Generator(device="cuda").manual_seed(3)
    first = torch.randint(0, n, (m,), generator=g, device="cuda")
    # column 11 is observed by the last 700 applications only: a column below the split length
    first = torch.where(first == n - 1, 0, first)
    cnt = torch.ones(m, dtype=torch.int64, device="cuda")
    cnt[-700:] = 2
    rp = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(cnt, 0, out=rp[1:])
    col = torch.full((int(rp[-1]),), n - 1, dtype=torch.int32, device="cuda")
    col[rp[:-1]] = first.to(torch.int32)
    val = 0.4 + 0.6 * torch.rand(col.numel(), generator=g, device="cuda")
    U = torch.zeros((m, k), device="cuda")
    V = 0.3 * torch.randn((n, k), generator=g, device="cuda")
    ctx = native.Context(0)
    try:
        native.open_fit(ctx, rp, col, val, U, V, LAM, 1, weighted=False)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    rows = torch.repeat_interleave(torch.arange(m, device="cuda"), cnt)
    for j in range(n):
        pick = torch.nonzero(col == j).flatten()
        u = U[rows[pick]].double()
        A = (u.T @ u).cpu().numpy() + LAM * np.eye(k)
        b = (u.T @ val[pick].double()).cpu().numpy()
        # the rows of U lie along the n directions of V0, so A is close to singular beside lambda: the
        # residual is what float32 sums and an LDL^T keep small
        e = np.linalg.norm(A @ V[j].double().cpu().numpy() - b) / np.linalg.norm(b)
        print("column %d of %d entries: residual %.2e" % (j, len(pick), e))
        assert e <= 1e-4
