"""Split-K parts of many thousand entries: the right-hand side, like the Gram matrix, is summed in
pieces of 1024 entries, so its error does not grow with the part.

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
