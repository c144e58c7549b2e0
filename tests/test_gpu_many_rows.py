"""More rows than one launch's threads can cover (a grid holds fewer than 2^32): the column view past
2^29 rows and the surrogate's forward pass past 2^28, of which only a few hold entries, and the NCF
model's gradient with 2^27 applications and more."""
import numpy as np
import pytest
import torch

from paper_2508_07605_amd import native, synth

pytestmark = pytest.mark.gpu


def row_pointers(m, rows):
    """Row pointers of m rows of which `rows` (ascending) hold one entry each."""
    rp = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    for e, i in enumerate(rows):
        rp[i + 1:] = e + 1
    return rp


def test_column_view():
    m, n = 2 ** 29 + 128 * 8200 + 5, 5
    rows = [0, 127, 128, 2 ** 28 - 1, 2 ** 28, 2 ** 28 + 127, 2 ** 29 - 1, 2 ** 29, 2 ** 29 + 128 * 8192, m - 1]
    col = np.array([4, 0, 4, 2, 4, 2, 0, 0, 2, 4], np.int32)
    val = np.arange(1, 11, dtype=np.float32)
    ctx = native.Context(0)
    try:
        cp, ri, cv = native.open_csr_to_csc(ctx, row_pointers(m, rows), torch.from_numpy(col).cuda(),
                                            torch.from_numpy(val).cuda(), n)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    order = np.lexsort((rows, col))
    assert cp.cpu().tolist() == [0, 3, 3, 6, 6, 10]
    assert np.array_equal(ri.cpu().numpy(), np.array(rows)[order])
    assert np.array_equal(cv.cpu().numpy(), val[order])


def test_forward():
    """Every row's output is, bit for bit, that of the same row in a small batch."""
    m, n, k = 2 ** 28 + 1001, 40, 8
    rows = [0, 5, 2 ** 26 - 1, 2 ** 26, 2 ** 27 + 3, 2 ** 28 - 1, 2 ** 28, 2 ** 28 + 1000]
    r = np.random.default_rng(4)
    col = torch.from_numpy(r.integers(0, n, size=len(rows)).astype(np.int32)).cuda()
    val = torch.from_numpy(r.uniform(0.4, 1.0, size=len(rows)).astype(np.float32)).cuda()
    ctx = native.Context(0)
    net = native.Surrogate(ctx, n, k, seed=2)
    try:
        out = torch.full((m, k), 7.0, device="cuda")
        net.forward(row_pointers(m, rows), col, val, out)
        few = net.forward(row_pointers(len(rows) + 1, range(len(rows))), col, val)
        torch.cuda.synchronize()
    finally:
        net.close()
        ctx.close()
    assert torch.equal(out[rows], few[:-1])
    same = (out == few[-1]).all(dim=1)
    same[rows] = True
    assert bool(same.all())


def test_ncf_gradient():
    """The gradient of a batch of a few applications out of many: theirs and the network's bit for
    bit as in a model of those applications alone, zero for the others."""
    m, n, d = 2 ** 27 + 4096, 3, 32
    apps = [m - 1, 17, 2 ** 27, 2 ** 27 - 1]
    p = synth.ncf_params(3, n, seed=1)
    S = p.pop("S")
    E = np.random.default_rng(6).normal(size=(len(apps), d)).astype(np.float32)
    few = torch.from_numpy(native.ncf_pack(E, S, p)).cuda()
    rest = few.numel() - len(apps) * d
    many = torch.zeros(m * d + rest, device="cuda")
    many[m * d:] = few[len(apps) * d:]
    many[:m * d].view(m, d)[apps] = torch.from_numpy(E).cuda()
    R = torch.full((m, n), 0.7, device="cuda")
    ctx = native.Context(0)
    try:
        loss, g = native.open_ncf_loss_grad(ctx, R, many, torch.tensor(apps, device="cuda"))
        want_loss, want = native.open_ncf_loss_grad(ctx, R[:len(apps)].contiguous(), few,
                                                    torch.arange(len(apps), device="cuda"))
    finally:
        ctx.close()
    assert loss == want_loss
    assert np.array_equal(g[m * d:], want[len(apps) * d:]) and want[len(apps) * d:].any()
    gE = g[:m * d].reshape(m, d)
    assert np.array_equal(gE[apps], want[:len(apps) * d].reshape(-1, d))
    gE[apps] = 0.0
    for a in range(0, m, 2 ** 22):
        assert not gE[a:a + 2 ** 22].any()
