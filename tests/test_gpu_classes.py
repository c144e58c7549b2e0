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
