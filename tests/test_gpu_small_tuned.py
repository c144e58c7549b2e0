"""Which kernels a small batch runs in a context whose tuning table is not the default: at rank 32 the
launch mode decides (merged launches do not read the class groups' entries, so tuning on a large
batch does not cost the one launch), with one launch per class group the kernels that the table
names run; the outputs are the default context's, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2508_07605_amd import native

pytestmark = pytest.mark.gpu


def run(table, k):
    r = np.random.default_rng(k)
    n, m = 480, 500
    counts = r.integers(0, 60, size=m)
    rp = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    col = np.concatenate([np.sort(r.choice(n, size=c, replace=False)) for c in counts]).astype(np.int32)
    val = r.uniform(0.4, 1.0, size=len(col)).astype(np.float32)
    V = (0.3 * r.normal(size=(n, k))).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ctx = native.Context(0)
    try:
        if table is not None:
            ctx.tune_set(k, table)
        ctx.profile(True)
        U = native.open_foldin(ctx, dev(V), dev(rp), dev(col), dev(val), 0.05, True)
        names = set(ctx.profile_read())
    finally:
        ctx.close()
    return U.cpu().numpy(), names


def test_rank_32_follows_the_launch_mode():
    groups = [name for name, _ in native.open_tune_info(32)]
    assert groups[-1] == "ridge_k32_launch"
    want, names = run(None, 32)
    assert names == {"foldin_small_k32"}
    tuned = [1, 1, 1, 0, 1, 1, 0, 0, 0]
    U, names = run(tuned + [0], 32)
    assert names == {"foldin_small_k32"} and np.array_equal(U, want)
    U, names = run(tuned + [1], 32)
    assert "foldin_small_k32" not in names and "ridge_k32_d4" in names
    assert np.abs(U - want).max() <= 1e-4 * np.abs(want).max()


@pytest.mark.parametrize("k", [8, 16])
def test_other_ranks_follow_the_table(k):
    ng = len(native.open_tune_info(k))
    assert run([0] * ng, k)[1] == {"foldin_small_k%d" % k}
    _, names = run([1] + [0] * (ng - 1), k)
    assert "ridge_k%d_d4" % k in names and "foldin_small_k%d" % k not in names
