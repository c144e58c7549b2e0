"""The two-launch training steps at the edges of its tiles and rules: batches around a tile of 16
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



def bf16(x):
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(torch.bfloat16).double().numpy()


def ncf_rounded_gradients(E, S, p, apps, R):
    """The batch's loss and gradients in float64 with every product's operands rounded to
    bfloat16 where the kernels round them.  (Against unrounded products a gradient of a small
    batch is off by the share of pre-activations that the rounding moves across SELU's kink.)"""
    from oracle.ncf import selu, selu_grad
    G, n = len(apps), S.shape[0]
    X = bf16(np.concatenate([np.repeat(E[apps], n, 0), np.tile(S, (G, 1))], 1))
    W1, W2, w3 = bf16(p["W1"]), bf16(p["W2"]), bf16(p["w3"])
    z1 = X @ W1.T + p["b1"]
    h1 = bf16(selu(z1))
    z2 = h1 @ W2.T + p["b2"]
    h2 = bf16(selu(z2))
    d = h2 @ w3 + p["b3"] - R[apps].reshape(-1).astype(np.float64)
    dy = 2.0 * d / d.size
    d2 = bf16(dy)[:, None] * w3 * selu_grad(z2)
    d1 = (bf16(d2) @ W2) * selu_grad(z1)
    dX = (bf16(d1) @ W1).reshape(G, n, 64)
    gE = np.zeros(E.shape)
    gE[apps] = dX[:, :, :32].sum(1)
    g = dict(E=gE, S=dX[:, :, 32:].sum(0), W1=bf16(d1).T @ X, b1=d1.sum(0), W2=bf16(d2).T @ h1, b2=d2.sum(0),
             w3=bf16(dy) @ h2, b3=np.array([dy.sum()]))
    return float(np.mean(d * d)), g


# NCF: batches of G applications x n settings around a tile of 16 or 32 rows and the switch
# between them, more settings than one pass of the embedding sums holds (1024), one
# application.  Tolerance: float32 accumulation moves a value by about 64 2^-24 relative, which
# carries about one value in a thousand across a bfloat16 rounding boundary (2^-8 relative):
# 1e-4 in a tensor's Frobenius norm; 1e-3 leaves room for small tensors.
@pytest.mark.parametrize("m_off,n,G", [(1, 1, 1), (5, 33, 3), (40, 31, 1), (16, 256, 16), (9, 480, 9), (3, 1025, 2),
                                       (2, 2100, 2)])
def test_ncf_gradients_at_tile_edges(ctx, m_off, n, G):
    r = np.random.default_rng([m_off, n, G])
    R = (3.0 + r.random((m_off, n))).astype(np.float32)
    p = synth.ncf_params(3, n, seed=2)
    S = p.pop("S")
    E = (0.3 * r.standard_normal((m_off, 32))).astype(np.float32)
    flat = dev(native.ncf_pack(E, S, p))
    apps = r.permutation(m_off)[:G].astype(np.int64)
    loss, g = native.open_ncf_loss_grad(ctx, dev(R), flat, dev(apps))
    Lr, gr = ncf_rounded_gradients(E, S, p, apps, R)
    gE, gS, gnet = native.ncf_unpack(g, m_off, n)
    errs = {"E": fro(gE, gr["E"]), "S": fro(gS, gr["S"])}
    errs.update({k: fro(v, gr[k]) for k, v in gnet.items()})
    print("NCF %d x %d, batch %d: loss %.6g vs %.6g, gradients %s"
          % (m_off, n, G, loss, Lr, {k: "%.1e" % v for k, v in errs.items()}))
    assert abs(loss - Lr) <= 1e-3 * Lr
    assert max(errs.values()) <= 1e-3
    assert not gE[np.setdiff1d(np.arange(m_off), apps)].any()
