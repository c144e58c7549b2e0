"""The two-launch training step at the edges of its tiles and rules: batches around a tile of 16
or 32 rows and around the switch between them, batch slices with a remainder, few slices with
several output tiles per block (wide inputs, large batches), many short slices (narrow output
layers), inputs that are no multiple of a tile, rows of more than 64 entries.

Tolerance: the products take operands rounded to bfloat16 (relative error at most 2^-9 each), so
a gradient tensor is within 1e-2 relative Frobenius of the float64 oracle on the same rounded
weights, the bound of the existing gradient tests."""
import numpy as np
import pytest
import torch

from oracle import mlp as omlp
from paper_2508_07605_amd import native, synth

pytestmark = pytest.mark.gpu
H = 256
TOL = 1e-2


@pytest.fixture(scope="module")
def ctx():
    c = native.Context(0)
    yield c
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def fro(a, b):
    return np.linalg.norm(np.asarray(a, np.float64) - b) / max(np.linalg.norm(b), 1e-300)


def batch(B, n, k, longest, seed):
    r = np.random.default_rng([B, n, k, seed])
    counts = r.integers(0, min(24, n) + 1, size=B)
    counts[-1] = longest
    rp = np.zeros(B + 1, np.int64)
    rp[1:] = np.cumsum(counts)
    col = np.concatenate([np.sort(r.choice(n, size=c, replace=False)) for c in counts]).astype(np.int32)
    val = r.uniform(0.4, 1.0, size=int(rp[-1])).astype(np.float32)
    return rp, col, val, r.standard_normal((B, k)).astype(np.float32)


@pytest.mark.parametrize("B,n,k,longest", [
    (1, 33, 8, 33), (15, 480, 32, 70), (17, 50, 16, 50), (33, 120, 8, 64), (257, 480, 64, 65), (1000, 480, 32, 24),
    (4096, 120, 8, 24), (4097, 120, 32, 24), (4100, 1920, 64, 130)])
def test_gradients_at_tile_edges(ctx, B, n, k, longest):
    params = synth.mlp_init(3, (2 * n, H, H, k), seed=5)
    net = native.Surrogate(ctx, n, k, H, init=np.concatenate([p.ravel() for p in params]))
    rp, col, val, target = batch(B, n, k, longest, 1)
    loss, g = net.loss_grad(dev(rp), dev(col), dev(val), dev(target))
    Lr, gr = omlp.loss_and_grads(params, omlp.dense_input(rp, col, val, n), target.astype(np.float64))
    o, errs = 0, []
    for want in gr:
        errs.append(fro(g[o:o + want.size].reshape(want.shape), want))
        o += want.size
    print("B %d n %d k %d: loss %.6g vs %.6g, gradients %s" % (B, n, k, loss, Lr, ["%.1e" % e for e in errs]))
    assert abs(loss - Lr) <= TOL * Lr
    assert max(errs) <= TOL
    # the step on the same batch moves by the same gradient: Adam's first step is lr sign(g)
    w0 = net.get_weights()
    net.train_step(dev(rp), dev(col), dev(val), dev(target), None, 1e-3)
    moved = net.get_weights() - w0
    clear = np.abs(g) > 1e-3 * np.abs(g).max()
    assert np.abs(moved + 1e-3 * np.sign(g))[clear].max() <= 2e-5
    assert np.all(moved[g == 0] == 0)
    # and leaves every copy of the weights in step: the gradient of the moved network
    _, g1 = net.loss_grad(dev(rp), dev(col), dev(val), dev(target))
    fresh = native.Surrogate(ctx, n, k, H, init=net.get_weights())
    _, g2 = fresh.loss_grad(dev(rp), dev(col), dev(val), dev(target))
    assert np.array_equal(g1, g2)
    net.close()
    fresh.close()
