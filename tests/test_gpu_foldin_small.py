"""The one-launch fold-in of small batches against the bucketed path of large ones: the same rows
inside a batch too large for it give the same bits, whatever their neighbours, at every rank
it serves, for factors staged in LDS (n <= 512) and not, both weightings, every status, and at
the edges of its blocks (128 rows) and of the rule (one block per compute unit at rank 32)."""
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


def csr(r, counts, n):
    rp = np.zeros(len(counts) + 1, np.int64)
    rp[1:] = np.cumsum(counts)
    col = np.concatenate([np.sort(r.choice(n, size=c, replace=False)) for c in counts] or [np.zeros(0)])
    return rp, col.astype(np.int32), r.uniform(0.4, 1.0, size=int(rp[-1])).astype(np.float32)


def foldin(ctx, V, rp, col, val, lam, weighted, fn=native.open_foldin):
    st = torch.full((len(rp) - 1,), -7, dtype=torch.int32, device="cuda")
    U = torch.full((len(rp) - 1, V.shape[1]), 7.0, device="cuda")
    fn(ctx, dev(V), dev(rp), dev(col), dev(val), lam, weighted, U_out=U, row_status=st)
    torch.cuda.synchronize()
    return U.cpu().numpy(), st.cpu().numpy()


@pytest.mark.parametrize("k,n", [(8, 120), (8, 600), (16, 480), (16, 700), (32, 480), (32, 600), (32, 40)])
@pytest.mark.parametrize("weighted", [True, False])
def test_small_equals_large_batch(ctx, k, n, weighted):
    r = np.random.default_rng([k, n, int(weighted)])
    counts = np.concatenate([np.repeat(np.arange(0, min(n, 36) + 1), 3), r.integers(0, min(n, 200) + 1, size=150), [n]])
    r.shuffle(counts)
    rp, col, val = csr(r, counts, n)
    V = (0.3 * r.normal(size=(n, k))).astype(np.float32)
    busy = np.nonzero(counts > 2)[0]
    val[rp[busy[0]]] = np.nan           # a non-finite value
    val[rp[busy[1] + 1] - 1] = np.inf
    col[rp[busy[2]]] = n                # a column out of range
    col[rp[busy[3]] + 1] = -1
    reps = 1 + 2 * 128 * 256 // len(counts)  # beyond the rule of every rank on a card of 256 units
    big_rp = np.concatenate([[0], np.cumsum(np.tile(counts, reps))]).astype(np.int64)
    for lam in (0.05, 0.0):
        U, st = foldin(ctx, V, rp, col, val, lam, weighted)
        Ub, stb = foldin(ctx, V, big_rp, np.tile(col, reps), np.tile(val, reps), lam, weighted)
        Ub, stb = Ub.reshape(reps, len(counts), k), stb.reshape(reps, len(counts))
        assert np.array_equal(st, stb[0]) and np.array_equal(st, stb[-1])
        assert np.array_equal(U, Ub[0]) and np.array_equal(U, Ub[-1])
        Un, stn = foldin(ctx, V, rp, col, val, lam, weighted, native.open_foldin_noalloc)
        assert np.array_equal(U, Un) and np.array_equal(st, stn)
    ok = np.ones(len(counts), bool)
    ok[busy[:4]] = False
    ref, ref_st = oracle.ridge_rows(rp, np.clip(col, 0, n - 1), np.nan_to_num(val, posinf=0.5), V, 0.05, weighted)
    U, st = foldin(ctx, V, rp, col, val, 0.05, weighted)
    assert np.array_equal(st[ok], ref_st[ok]) and np.array_equal(st[busy[:4]], [3, 3, 5, 5])
    nrm = np.maximum(np.linalg.norm(ref[ok], axis=1), 1e-30)
    assert (np.linalg.norm(U[ok] - ref[ok], axis=1) / np.where(counts[ok] > 0, nrm, 1.0)).max() <= 1e-4


@pytest.mark.parametrize("m", [1, 15, 127, 128, 129, 1000, 32767, 32768, 32769])
def test_block_and_rule_edges(ctx, m):
    r = np.random.default_rng(m)
    n, k = 480, 32
    counts = r.integers(0, 28, size=m)
    cols = np.argsort(r.random((64, n)), axis=1)
    rp = np.zeros(m + 1, np.int64)
    rp[1:] = np.cumsum(counts)
    col = np.concatenate([np.sort(cols[i % 64][:c]) for i, c in enumerate(counts)] or [np.zeros(0)]).astype(np.int32)
    val = r.uniform(0.4, 1.0, size=max(int(rp[-1]), 1)).astype(np.float32)[:int(rp[-1])]
    V = (0.3 * r.normal(size=(n, k))).astype(np.float32)
    if len(col) == 0:
        col, val = np.zeros(1, np.int32), np.zeros(1, np.float32)
    U, st = foldin(ctx, V, rp, col, val, 0.05, False)
    sample = np.unique(np.concatenate([np.arange(min(m, 300)), np.arange(max(0, m - 300), m)]))
    ref, ref_st = oracle.ridge_subset(sample, rp, col, val, V, 0.05, False)
    assert np.array_equal(st[sample], ref_st)
    nrm = np.linalg.norm(ref, axis=1)
    assert (np.linalg.norm(U[sample] - ref, axis=1) / np.where(nrm > 0, nrm, 1.0)).max() <= 1e-4
    assert (st != -7).all() and np.isfinite(U).all() and (U[counts == 0] == 0).all()
