"""Length classes of the primal ridge solves (four per doubling): rows at both sides of every
class boundary and of the split-K length, in batches large enough for the bucketed path, at every
rank; per-row error against the float64 oracle at most 1e-4 and statuses equal."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_07605_amd import native

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("k,n", [(8, 480), (8, 1100), (16, 480), (16, 1100), (32, 480), (32, 700), (32, 1100), (64, 480),
                                 (64, 1100)])
def test_class_boundaries(k, n):
    r = np.random.default_rng([k, n])
    edges = {k, k + 1, 31, 32, 33, 64, 65, n}
    for octave in range(8):
        for sub in range(4):
            b = k * (4 + sub) * 2 ** octave // 4
            edges |= {b, b + 1, b + 2}
    if n >= 1024:
        edges |= {1023, 1024, 1025}
    counts = np.array(sorted(c for c in edges if 0 < c <= n))
    counts = np.concatenate([counts, np.zeros(2, np.int64), counts[::-1]])
    ctx = native.Context(0)
    try:
        pad = 0 if k == 64 or n >= 1024 else 2 * 128 * 256  # past the one-launch path of small batches
        allc = np.concatenate([counts, np.full(pad, 3, np.int64)])
        rp = np.zeros(len(allc) + 1, np.int64)
        rp[1:] = np.cumsum(allc)
        head = np.concatenate([np.sort(r.choice(n, size=c, replace=False)) for c in counts])
        tail = (np.arange(3)[None, :] * 7 + (np.arange(pad) % 400)[:, None]).ravel()
        col = np.concatenate([head, tail]).astype(np.int32)
        val = r.uniform(0.4, 1.0, size=len(col)).astype(np.float32)
        V = (0.3 * r.normal(size=(n, k))).astype(np.float32)
        st = torch.full((len(allc),), -7, dtype=torch.int32, device="cuda")
        U = native.open_foldin(ctx, dev(V), dev(rp), dev(col), dev(val), 0.05, True, row_status=st)
        torch.cuda.synchronize()
        U, st = U.cpu().numpy().astype(np.float64), st.cpu().numpy()
    finally:
        ctx.close()
    m = len(counts) + min(pad, 50)
    ref, ref_st = oracle.ridge_rows(rp[:m + 1], col[:rp[m]], val[:rp[m]], V, 0.05, True)
    assert np.array_equal(st[:m], ref_st) and (st[m:] == 0).all()
    nrm = np.linalg.norm(ref, axis=1)
    e = np.linalg.norm(U[:m] - ref, axis=1) / np.where(nrm > 0, nrm, 1.0)
    print("k %d n %d: max error %.2e" % (k, n, e.max()))
    assert e.max() <= 1e-4


@pytest.mark.parametrize("k,n", [(32, 480), (32, 700), (16, 480), (8, 480)])
def test_groups_handed_out(k, n):
    """More groups of primal rows than wavefronts on the card, of very different lengths: every row
    is solved once, and to the bits that it has in a batch small enough for one group each."""
    r = np.random.default_rng([k, n])
    m = 75_001
    counts = np.minimum(r.zipf(1.4, size=m) + k, n - 1).astype(np.int64)
    counts[r.integers(0, m, size=2000)] = r.integers(0, k, size=2000)  # some dual and empty rows
    rp = np.zeros(m + 1, np.int64)
    rp[1:] = np.cumsum(counts)
    start = r.integers(0, n, size=m)
    col = ((np.arange(rp[-1]) - np.repeat(rp[:-1], counts) + np.repeat(start, counts)) % n).astype(np.int32)
    val = r.uniform(0.4, 1.0, size=len(col)).astype(np.float32)
    V = dev((0.3 * r.normal(size=(n, k))).astype(np.float32))
    ctx = native.Context(0)
    try:
        def solve(a, b):
            st = torch.full((b - a,), -7, dtype=torch.int32, device="cuda")
            sl = slice(int(rp[a]), int(rp[b]))
            U = torch.full((b - a, k), float("nan"), device="cuda")
            native.open_foldin(ctx, V, dev(rp[a:b + 1] - rp[a]), dev(col[sl]), dev(val[sl]), 0.05, True, U_out=U,
                               row_status=st)
            return U.cpu(), st.cpu()

        U, st = solve(0, m)
        parts = [solve(a, min(a + 25_001, m)) for a in range(0, m, 25_001)]
    finally:
        ctx.close()
    assert torch.equal(U, torch.cat([p[0] for p in parts])) and torch.equal(st, torch.cat([p[1] for p in parts]))
    assert torch.equal(st == 0, torch.from_numpy(counts > 0))
