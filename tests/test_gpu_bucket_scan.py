"""Bucketing of more blocks of rows than the place kernel sums itself (512 of 2048 rows), with the scan
of each class in rounds of 4096 counts: the same rows, in the order of their groups or not, have
the bits that they have in small batches."""
import numpy as np
import pytest
import torch

from paper_2508_07605_amd import native

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [2048 * 512, 2048 * 512 + 1, 2048 * 4096 + 3])
def test_many_blocks(m):
    k, n = 8, 60
    g = torch.Generator(device="cuda").manual_seed(m)
    # kinds of rows: empty, dual, primal of several lengths; long stretches of one kind among them
    kinds = torch.tensor([0, 1, 4, 5, 8, 9, 17, 40], device="cuda")
    which = torch.randint(0, 8, (m,), generator=g, device="cuda")
    which[m // 3: m // 2] = 2
    cnt = kinds[which]
    rp = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(cnt, 0, out=rp[1:])
    nnz = int(rp[-1])
    rows = torch.repeat_interleave(torch.arange(m, device="cuda"), cnt, output_size=nnz)
    t = torch.arange(nnz, device="cuda") - rp[rows]
    shift = torch.randint(0, 20, (m,), generator=g, device="cuda")  # few rows differ: 8 x 20 of them
    col = (t + shift[rows]).to(torch.int32)
    val = 0.4 + 0.01 * ((t + 3 * shift[rows]) % 50).float()
    V = torch.from_numpy((0.3 * np.random.default_rng(1).normal(size=(n, k))).astype(np.float32)).cuda()
    ctx = native.Context(0)
    try:
        def solve(a, b):
            st = torch.full((b - a,), -7, dtype=torch.int32, device="cuda")
            e0, e1 = int(rp[a]), int(rp[b])
            U = torch.full((b - a, k), 7.0, device="cuda")
            native.open_foldin(ctx, V, rp[a:b + 1] - e0, col[e0:e1].contiguous(), val[e0:e1].contiguous(), 0.05, True,
                               U_out=U, row_status=st)
            return U, st

        U, st = solve(0, m)
        few, few_st = solve(0, 20_000)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    assert torch.equal(U[:20_000], few) and torch.equal(st[:20_000], few_st)
    # every other row against the first of its kind and shift
    key = which * 20 + shift
    first = torch.full((160,), -1, dtype=torch.int64, device="cuda")
    first[key[:20_000].flip(0)] = torch.arange(19_999, -1, -1, device="cuda")
    assert (first >= 0).all()
    assert torch.equal(U, U[first[key]]) and torch.equal(st, st[first[key]])
