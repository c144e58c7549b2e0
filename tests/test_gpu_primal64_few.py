"""Rank-64 rows of the primal form in batches of few such rows, which are solved one per wavefront, and
in large ones, four per wavefront: the same rows give the same bits in both, and agree with the
float64 oracle to 1e-4 (the bound of the other ridge tests), with every status, at both sides of
the rule (8 wavefronts on each of 256 compute units)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_07605_amd import native

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def foldin(ctx, V, rp, col, val, lam, weighted):
    st = torch.full((len(rp) - 1,), -7, dtype=torch.int32, device="cuda")
    U = native.open_foldin(ctx, V, dev(rp), dev(col), dev(val), lam, weighted,
                           U_out=torch.full((len(rp) - 1, 64), 7.0, device="cuda"), row_status=st)
    torch.cuda.synchronize()
    return U.cpu().numpy(), st.cpu().numpy()


@pytest.mark.parametrize("weighted", [True, False])
@pytest.mark.parametrize("n", [480, 1023, 1500])
def test_few_equals_many(n, weighted):
    k = 64
    r = np.random.default_rng([n, int(weighted)])
    longest = min(n, 1023)
    counts = np.concatenate([[33, 34, 63, 64, 65, 128, 255, 256, 257, 272, longest - 1, longest],
                             r.integers(33, longest + 1, size=30)])
    rp = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    col = np.concatenate([np.sort(r.choice(n, size=c, replace=False)) for c in counts]).astype(np.int32)
    val = r.uniform(0.4, 1.0, size=len(col)).astype(np.float32)
    V = (0.3 * r.normal(size=(n, k))).astype(np.float32)
    val[rp[15] + 20] = np.nan
    val[rp[16] + 1] = -np.inf
    col[rp[17]] = n
    col[rp[18 + 1] - 1] = -3
    reps = 1 + 2048 // len(counts)
    many_rp = np.concatenate([[0], np.cumsum(np.tile(counts, reps))]).astype(np.int64)
    ctx = native.Context(0)
    try:
        dV = dev(V)
        for lam in (0.05, 0.0):
            U, st = foldin(ctx, dV, rp, col, val, lam, weighted)
            Um, stm = foldin(ctx, dV, many_rp, np.tile(col, reps), np.tile(val, reps), lam, weighted)
            assert np.array_equal(st, stm[:len(st)]) and np.array_equal(st, stm[-len(st):])
            good = st == 0  # (a row refused at a pivot writes zeros in both)
            assert np.array_equal(U, Um[:len(st)]) and np.array_equal(U, Um[-len(st):]) and (U[~good] == 0).all()
        U, st = foldin(ctx, dV, rp, col, val, 0.05, weighted)
    finally:
        ctx.close()
    ok = np.ones(len(counts), bool)
    ok[15:19] = False
    assert np.array_equal(st[15:19], [3, 3, 5, 5])
    ref, ref_st = oracle.ridge_rows(rp, np.clip(col, 0, n - 1), np.nan_to_num(val, neginf=0.5), V, 0.05, weighted)
    assert np.array_equal(st[ok], ref_st[ok])
    e = np.linalg.norm(U[ok] - ref[ok], axis=1) / np.linalg.norm(ref[ok], axis=1)
    print("n %d: max error %.2e" % (n, e.max()))
    assert e.max() <= 1e-4


@pytest.mark.parametrize("m", [1, 2, 7, 255, 256, 257, 2047, 2048, 2049, 4097])
def test_rule_edges(m):
    """m rows of the class among other rows: all solved, once, to the bits of the first of their kind."""
    n, k = 200, 64
    r = np.random.default_rng(m)
    kinds = [(c, np.sort(r.choice(n, size=c, replace=False))) for c in (40, 33, 100, 5)]
    which = np.concatenate([np.arange(m) % 3, np.full(50, 3)])
    r.shuffle(which)
    counts = np.array([kinds[i][0] for i in which])
    rp = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    col = np.concatenate([kinds[i][1] for i in which]).astype(np.int32)
    val = (0.4 + 0.5 * np.sin(np.arange(n)) ** 2).astype(np.float32)[col]
    V = (0.3 * r.normal(size=(n, k))).astype(np.float32)
    ctx = native.Context(0)
    try:
        U, st = foldin(ctx, dev(V), rp, col, val, 0.05, True)
    finally:
        ctx.close()
    assert (st == 0).all()
    for i in range(4):
        rows = np.nonzero(which == i)[0]
        if len(rows):
            assert (U[rows] == U[rows[0]]).all()
            c = kinds[i][1]
            ref = np.linalg.solve(V[c].T.astype(np.float64) @ V[c] + 0.05 * len(c) * np.eye(k),
                                  V[c].T.astype(np.float64) @ val[rp[rows[0]]:rp[rows[0] + 1]])
            assert np.linalg.norm(U[rows[0]] - ref) <= 1e-4 * np.linalg.norm(ref)
