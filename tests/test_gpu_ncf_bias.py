"""NCF training batches of many rows, whose bias gradients are summed by a launch of their own: at both
sides of the rule (8192 rows, four applications), with slices of one and several groups of rows and a
last slice that is not full.  The gradients against float64 with the same bfloat16 roundings, to 1e-3 in
each tensor's Frobenius norm (float32 sums over B rows: about sqrt(B) 2^-24, and one value in a thousand
carried across a rounding boundary of 2^-8, as in the tests of small batches); twice the same bits."""
import numpy as np
import pytest
import torch

from paper_2508_07605_amd import native, synth
from test_gpu_train_step import fro, ncf_rounded_gradients

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,n", [(16, 512), (17, 483), (3, 2750), (4, 2049), (69, 119), (100, 480), (40, 1000)])
def test_gradients(G, n):
    m = G + 3
    r = np.random.default_rng([G, n])
    R = (3.0 + r.random((m, n))).astype(np.float32)
    p = synth.ncf_params(3, n, seed=2)
    S = p.pop("S")
    E = (0.3 * r.standard_normal((m, 32))).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    flat, apps = dev(native.ncf_pack(E, S, p)), r.permutation(m)[:G].astype(np.int64)
    ctx = native.Context(0)
    try:
        loss, g = native.open_ncf_loss_grad(ctx, dev(R), flat, dev(apps))
        loss2, g2 = native.open_ncf_loss_grad(ctx, dev(R), flat, dev(apps))
    finally:
        ctx.close()
    assert loss == loss2 and np.array_equal(g, g2)
    Lr, gr = ncf_rounded_gradients(E, S, p, apps, R)
    gE, gS, gnet = native.ncf_unpack(g, m, n)
    errs = {"E": fro(gE, gr["E"]), "S": fro(gS, gr["S"])}
    errs.update({k: fro(v, gr[k]) for k, v in gnet.items()})
    print("NCF %d x %d: loss %.6g vs %.6g, gradients %s" % (G, n, loss, Lr, {k: "%.1e" % v for k, v in errs.items()}))
    assert abs(loss - Lr) <= 1e-3 * Lr
    assert max(errs.values()) <= 1e-3
