"""Performance cases of the CF-completion library: what a user of it has it do, path by path.

Every case goes through the Python binding of the C ABI (paper_2508_07605_amd.native).  Inputs
follow the distributions of paper_2508_07605_amd.synth (the cap grids, the applications'
sensitivities, the observed sets, the noise), drawn on the GPU from the seed so that they are
quick to make.  listed() holds the sizes of the library's own configurations from the smallest
to the largest; draw() takes the ranges around them.  exact() evaluates the same definitions in
float64 with plain torch and numpy.
"""
import functools
import math

import numpy as np
import torch

from paper_2508_07605_amd import native, synth

NOISE = 0.02
LAM = 0.05
HIDDEN = 256
NCF_D, NCF_H = 32, 64


# ------------------------------------------------------------------------------- the cases
def listed():
    return [
        # online phase, one arrival: 16 new applications with 6 profiled settings each against a
        # small grid (the "tiny" configuration) -- launch latency
        dict(name="foldin_16", path="foldin", m=16, n_cpu=12, n_gpu=10, k=8, counts="uniform", lo=6, hi=6,
             weighted=True, entry="foldin"),
        # online phase, an ordinary batch of arrivals on the 480-setting grid
        dict(name="foldin_4099", path="foldin", m=4099, n_cpu=24, n_gpu=20, k=32, counts="uniform", lo=4, hi=24,
             weighted=False, entry="foldin"),
        # the headline workload: 1M new applications with 4..24 observed settings
        dict(name="foldin_1m", path="foldin", m=1_000_000, n_cpu=24, n_gpu=20, k=32, counts="uniform", lo=4, hi=24,
             weighted=False, entry="foldin"),
        # offline phase: the ALS-WR fit of 200k applications x 480 settings (configuration "fit")
        dict(name="fit_200k", path="fit", m=200_003, n_cpu=24, n_gpu=20, k=32, zipf=1.2, sweeps=5),
        # offline phase on the large grid: 48 x 40 caps, rank 64, a quarter of the 2M applications
        dict(name="fit_large", path="fit", m=500_009, n_cpu=48, n_gpu=40, k=64, zipf=1.6931, sweeps=3),
        # selection of the cap pair over all 1920 settings (prediction fused with Algorithm 2)
        dict(name="predict_1m_k64", path="predict", m=1_000_003, n_cpu=48, n_gpu=40, k=64, gamma=0.05, want_p=False),
        # surrogate fold-in with the ridge fallback on about a fifth of the rows
        dict(name="surrogate_1m", path="surrogate", m=1_000_000, n_cpu=24, n_gpu=20, k=32, tau=0.085),
        # surrogate training: two epochs of 48 Adam steps at the configuration's batch
        dict(name="surrogate_train", path="surrogate_train", m=200_003, n_cpu=24, n_gpu=20, k=32, batch=4096, epochs=2),
        # NCF fold-in of new applications: 30 gradient steps each
        dict(name="ncf_foldin", path="ncf", m=65_536, n_cpu=24, n_gpu=20, lo=4, hi=24, steps=30),
        # NCF offline training: one epoch over 1024 dense applications in batches of 8
        dict(name="ncf_train", path="ncf_train", m=1024, n_cpu=24, n_gpu=20, group=8, epochs=1),
        # Algorithm 1 over recorded power traces: 10 minutes at 0.2 s, 25-reading window
        dict(name="phase_65536", path="phase", m=65_536, length=3000, window=25),
        # offline predictor over all profiled runs of the headline workload
        dict(name="predictor_14m", path="predictor", m=14_000_003),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


GRIDS = ((12, 10), (24, 20), (48, 40))


def draw(rng):
    path = rng.choice(("foldin", "foldin", "fit", "predict", "surrogate", "surrogate_train", "ncf", "ncf_train", "phase",
                       "predictor"))
    nc, ng = rng.choice(GRIDS)
    n = nc * ng
    if path == "foldin":
        if rng.random() < 0.7:
            lo = rng.randint(1, 12)
            c = dict(path=path, m=_log_int(rng, 16, 1_000_000), n_cpu=nc, n_gpu=ng, k=rng.choice((8, 16, 32, 64)),
                     counts="uniform", lo=lo, hi=lo + rng.randint(0, 20))
        else:  # long-tailed counts up to the whole grid
            c = dict(path=path, m=_log_int(rng, 16, 150_000), n_cpu=nc, n_gpu=ng, k=rng.choice((8, 16, 32, 64)),
                     counts="zipf", zipf=rng.uniform(1.2, 1.7), lo=3, hi=n)
        c.update(weighted=rng.random() < 0.5, entry="foldin" if n >= 1024 else rng.choice(("foldin", "noalloc")))
        return c
    if path == "fit":
        return dict(path=path, m=_log_int(rng, 64, 200_000), n_cpu=nc, n_gpu=ng,
                    k=rng.choice((8, 16, 32, 64)) if n > 120 else rng.choice((8, 16)), zipf=rng.uniform(1.2, 1.7),
                    sweeps=rng.randint(1, 3))
    if path == "predict":
        want_p = rng.random() < 0.25
        return dict(path=path, m=_log_int(rng, 16, 100_000 if want_p else 1_000_000), n_cpu=nc, n_gpu=ng,
                    k=rng.choice((8, 16, 32, 64)), gamma=rng.choice((0.02, 0.05, 0.1)), want_p=want_p)
    if path == "surrogate":
        nc, ng, k = rng.choice(((24, 20, 32), (24, 20, 16), (48, 40, 64)))
        return dict(path=path, m=_log_int(rng, 100, 500_000 if k == 64 else 1_000_000), n_cpu=nc, n_gpu=ng, k=k,
                    tau=rng.choice((0.03, 0.06, 0.085)))
    if path == "surrogate_train":
        nc, ng, k = rng.choice(((24, 20, 32), (24, 20, 16), (12, 10, 8)))
        b = rng.choice((512, 1000, 2048, 4096))
        return dict(path=path, m=b * rng.randint(8, 40) + rng.randint(0, b - 1), n_cpu=nc, n_gpu=ng, k=k, batch=b,
                    epochs=rng.randint(1, 2))
    if path == "ncf":
        lo = rng.randint(1, 10)
        return dict(path=path, m=_log_int(rng, 16, 65_536), n_cpu=nc, n_gpu=ng, lo=lo, hi=lo + rng.randint(0, 14),
                    steps=rng.randint(5, 30))
    if path == "ncf_train":
        nc, ng = rng.choice(GRIDS[:2])
        g = rng.randint(2, 16)
        return dict(path=path, m=g * rng.randint(10, 60), n_cpu=nc, n_gpu=ng, group=g, epochs=1)
    if path == "phase":
        return dict(path=path, m=_log_int(rng, 16, 65_536), length=rng.randint(300, 3000), window=rng.randint(5, 50))
    return dict(path=path, m=_log_int(rng, 100, 14_000_000))


# ------------------------------------------------------------------------------- inputs
def _dev():
    return torch.device("cuda", torch.cuda.current_device())


@functools.lru_cache(maxsize=None)
def _ctx():
    return native.Context(torch.cuda.current_device())


def _gen(seed, tag):
    return torch.Generator(device=_dev()).manual_seed(1_000_003 * int(seed) + tag)


@functools.lru_cache(maxsize=None)
def _grid(n_cpu, n_gpu):
    return synth.cap_grid(n_cpu, n_gpu)


@functools.lru_cache(maxsize=None)
def _setting_factors(n_cpu, n_gpu, k):
    return synth.setting_factors(3, _grid(n_cpu, n_gpu), k, m_ref=1024)


def _uniform(g, size, lo=0.0, hi=1.0, dtype=torch.float64):
    return lo + (hi - lo) * torch.rand(size, generator=g, device=_dev(), dtype=dtype)


def _apps(g, m):
    """beta ~ Beta(2, 2) (the median of three uniforms), exponents ~ U(0.3, 1)."""
    beta = _uniform(g, (m, 3)).median(dim=1).values
    return beta, _uniform(g, m, 0.3, 1.0), _uniform(g, m, 0.3, 1.0)


def _truth(apps, grid, rows, cols):
    beta, gc, gg = (a[rows] for a in apps)
    c = torch.from_numpy(grid.cpu_w.max() / grid.cpu_w).to(_dev())[cols]
    w = torch.from_numpy(grid.gpu_w.max() / grid.gpu_w).to(_dev())[cols]
    return 1.0 / (beta * c ** gc + (1.0 - beta) * w ** gg)


def _truth_dense(apps, grid):
    m = apps[0].numel()
    r = torch.arange(m, device=_dev())[:, None].expand(m, grid.n)
    c = torch.arange(grid.n, device=_dev())[None, :].expand(m, grid.n)
    return _truth(apps, grid, r, c)


def _pmf(case, n):
    """(counts, probabilities) of a row's observed entries."""
    if case.get("counts", "zipf") == "uniform" or "zipf" not in case:
        ks = np.arange(min(case.get("lo", 4), n), min(case.get("hi", 24), n) + 1)
        return ks, np.full(len(ks), 1.0 / len(ks))
    ks = np.arange(3, n + 1)
    p = ks.astype(np.float64) ** -float(case["zipf"])
    return ks, p / p.sum()


def _rows(case, seed, grid):
    """CSR rows: (row_ptr int64, col int32, val float32).  A row's observed set is a run of a
    random permutation of the settings (one of 1024), sorted."""
    m, n, g = case["m"], grid.n, _gen(seed, 1)
    apps = _apps(g, m)
    ks, p = _pmf(case, n)
    cdf = torch.from_numpy(np.cumsum(p)).to(_dev())
    pick = torch.searchsorted(cdf, _uniform(g, m)).clamp_(max=len(ks) - 1)
    cnt = torch.from_numpy(ks).to(_dev())[pick]
    row_ptr = torch.zeros(m + 1, dtype=torch.int64, device=_dev())
    torch.cumsum(cnt, 0, out=row_ptr[1:])
    nnz = int(row_ptr[-1])
    perms = torch.rand((1024, n), generator=g, device=_dev()).argsort(dim=1)
    which = torch.randint(0, 1024, (m,), generator=g, device=_dev())
    start = torch.randint(0, n, (m,), generator=g, device=_dev())
    rows = torch.repeat_interleave(torch.arange(m, device=_dev()), cnt, output_size=nnz)
    t = torch.arange(nnz, device=_dev()) - row_ptr[rows]
    key = rows * n + perms[which[rows], (start[rows] + t) % n]
    del t
    col = torch.sort(key).values - rows * n
    val = _truth(apps, grid, rows, col)
    val = val * (1.0 + NOISE * torch.randn(nnz, generator=g, device=_dev(), dtype=torch.float64))
    return row_ptr, col.to(torch.int32), val.to(torch.float32)


def _init_factors(case, seed, n):
    g = _gen(seed, 2)
    U = 0.1 * torch.randn((case["m"], case["k"]), generator=g, device=_dev())
    V = 0.1 * torch.randn((n, case["k"]), generator=g, device=_dev())
    return U, V


@functools.lru_cache(maxsize=None)
def _prototypes(n_cpu, n_gpu, k):
    """Factors of 512 applications that predict their noiseless truth (least squares)."""
    grid = _grid(n_cpu, n_gpu)
    T = synth.truth_dense(synth.draw_apps(synth.rng(3, synth.S_EVAL, 0), 512), grid)
    V = _setting_factors(n_cpu, n_gpu, k).astype(np.float64)
    return np.linalg.lstsq(V, T.T, rcond=None)[0].T


def _bf16(x):
    return x.to(torch.float32).to(torch.bfloat16).to(torch.float64)


def _gelu(z):
    return 0.5 * z * (1.0 + torch.erf(z / math.sqrt(2.0)))


def _dense_x(row_ptr, col, val, n, a, b):
    """Rows a..b of the masked profile vectors [r * mask ; mask], float64."""
    e0, e1 = int(row_ptr[a]), int(row_ptr[b])
    cnt = row_ptr[a + 1:b + 1] - row_ptr[a:b]
    rows = torch.repeat_interleave(torch.arange(b - a, device=col.device), cnt, output_size=e1 - e0)
    X = torch.zeros((b - a, 2 * n), dtype=torch.float64, device=col.device)
    c = col[e0:e1].long()
    X[rows, c] = val[e0:e1].double()
    X[rows, n + c] = 1.0
    return X


def _net_split(w, n, k):
    o, out = 0, []
    for shape in ((HIDDEN, 2 * n), (HIDDEN,), (HIDDEN, HIDDEN), (HIDDEN,), (k, HIDDEN), (k,)):
        c = int(np.prod(shape))
        out.append(w[o:o + c].reshape(shape))
        o += c
    return out


@functools.lru_cache(maxsize=2)
def _surrogate_weights(n_cpu, n_gpu, k):
    """A network that imitates the fold-in: random hidden layers, the output layer fitted by
    ridge regression to the fold-ins of 16384 applications (a training run takes too long
    here).  Host float32 vector in the library's packing."""
    grid = _grid(n_cpu, n_gpu)
    n = grid.n
    case = dict(m=16384, lo=4, hi=24, counts="uniform", k=k, n_cpu=n_cpu, n_gpu=n_gpu, weighted=False)
    rp, col, val = _rows(case, 77, grid)
    F = torch.from_numpy(_setting_factors(n_cpu, n_gpu, k)).to(_dev())
    target = _exact_ridge(rp, col, val, F, LAM, False)
    w = torch.from_numpy(np.concatenate([x.ravel() for x in synth.mlp_init(3, (2 * n, HIDDEN, HIDDEN, k))])).to(_dev())
    W1, b1, W2, b2, W3, b3 = _net_split(w, n, k)
    W1 *= 4.0  # a row observes a few settings out of n: the hidden units need a spread of values
    W2 *= 2.0
    H = []
    for a in range(0, case["m"], 8192):
        X = _dense_x(rp, col, val, n, a, min(a + 8192, case["m"]))
        H.append(_gelu(_bf16(_gelu(X @ _bf16(W1).T + b1.double())) @ _bf16(W2).T + b2.double()))
    H = torch.cat(H)
    A = torch.cat([H, torch.ones_like(H[:, :1])], 1)
    G = A.T @ A + 1e-3 * torch.eye(HIDDEN + 1, dtype=torch.float64, device=_dev())
    sol = torch.from_numpy(np.linalg.solve(G.cpu().numpy(), (A.T @ target).cpu().numpy())).to(_dev())
    W3.copy_(sol[:HIDDEN].T)
    b3.copy_(sol[HIDDEN])
    return w.cpu().numpy()


def _initial_weights(case, n, seed):
    k = case["k"]
    return np.concatenate([x.ravel() for x in synth.mlp_init(3, (2 * n, HIDDEN, HIDDEN, k), seed=seed)])


def _caps(grid):
    return (torch.from_numpy(grid.cpu_w.astype(np.float32)).to(_dev()),
            torch.from_numpy(grid.gpu_w.astype(np.float32)).to(_dev()))


def prepare(case, seed):
    path = case["path"]
    s = dict(case=case, path=path, ctx=_ctx())
    if path == "phase":
        s["power"] = _power(case, seed)
        return s
    if path == "predictor":
        s["X"] = _features(case, seed)
        s["params"] = {k: torch.from_numpy(v).to(_dev())
                       for k, v in synth.predictor_params(3, _grid(24, 20), seed=seed).items()}
        return s
    grid = _grid(case["n_cpu"], case["n_gpu"])
    n = grid.n
    if path in ("foldin", "fit", "surrogate", "surrogate_train", "ncf"):
        s["row_ptr"], s["col"], s["val"] = _rows(case, seed, grid)
    if path in ("foldin", "surrogate", "surrogate_train", "predict"):
        s["F"] = torch.from_numpy(_setting_factors(case["n_cpu"], case["n_gpu"], case["k"])).to(_dev())
    if path == "foldin" and case["entry"] == "noalloc":
        s["U"] = torch.empty((case["m"], case["k"]), device=_dev())
    if path == "fit":
        s["U0"], s["V0"] = _init_factors(case, seed, n)
    if path == "predict":
        g = _gen(seed, 3)
        proto = torch.from_numpy(_prototypes(case["n_cpu"], case["n_gpu"], case["k"])).to(_dev())
        pick = torch.randint(0, proto.shape[0], (case["m"],), generator=g, device=_dev())
        noise = torch.randn((case["m"], case["k"]), generator=g, device=_dev())
        s["U"] = (proto[pick] + 0.01 * noise).to(torch.float32)
        s["cap_cpu"], s["cap_gpu"] = _caps(grid)
        s["base"] = grid.base
    if path == "surrogate":
        w = _surrogate_weights(case["n_cpu"], case["n_gpu"], case["k"])
        s["net"] = native.Surrogate(_ctx(), n, case["k"], HIDDEN, init=w)
    if path == "surrogate_train":
        s["target"] = _exact_ridge(s["row_ptr"], s["col"], s["val"], s["F"], LAM, False).to(torch.float32)
        s["w0"] = _initial_weights(case, n, seed)
        s["net"] = native.Surrogate(_ctx(), n, case["k"], HIDDEN, init=s["w0"])
        s["seed"] = seed
    if path == "ncf":
        p = synth.ncf_params(3, n, seed=seed)
        s["S"] = torch.from_numpy(p.pop("S")).to(_dev())
        s["params"] = {k: torch.from_numpy(v).to(_dev()) for k, v in p.items()}
    if path == "ncf_train":
        s["R"] = _truth_dense(_apps(_gen(seed, 1), case["m"]), grid).to(torch.float32)
        p = synth.ncf_params(3, n, seed=seed)
        flat = native.ncf_pack(np.zeros((case["m"], NCF_D)), p.pop("S"), p)
        s["p0"] = torch.from_numpy(flat).to(_dev())
        s["p"] = torch.empty_like(s["p0"])
        s["seed"] = seed
    return s


def _power(case, seed):
    m, L, g = case["m"], case["length"], _gen(seed, 4)
    start = torch.randint(0, L, (m, 1), generator=g, device=_dev())
    start = torch.where(_uniform(g, (m, 1)) < 0.1, L, start)
    lo, hi = _uniform(g, (m, 1), 25.0, 55.0, torch.float32), _uniform(g, (m, 1), 120.0, 280.0, torch.float32)
    on = torch.arange(L, device=_dev())[None, :] >= start
    p = torch.where(on, hi, lo) + 3.0 * torch.randn((m, L), generator=g, device=_dev())
    dip = on & (torch.rand((m, L), generator=g, device=_dev()) < 0.01)
    return torch.where(dip, _uniform(g, (m, L), 20.0, 59.0, torch.float32), p)


def _features(case, seed):
    m, grid, g = case["m"], _grid(24, 20), _gen(seed, 5)
    X = torch.empty((m, 7), device=_dev())
    j = torch.randint(0, grid.n, (m,), generator=g, device=_dev())
    for f, caps in enumerate(_caps(grid)):
        X[:, f] = caps[j]
    for f, (lo, hi) in enumerate(synth.COUNTER_RANGES):
        X[:, 2 + f] = _uniform(g, m, lo, hi, torch.float32)
    return X


# ------------------------------------------------------------------------------- one pass
def run(s):
    case, ctx = s["case"], s["ctx"]
    path = s["path"]
    if path == "foldin":
        status = torch.empty(case["m"], dtype=torch.int32, device=s["F"].device)
        if case["entry"] == "noalloc":
            native.open_foldin_noalloc(ctx, s["F"], s["row_ptr"], s["col"], s["val"], LAM, case["weighted"], s["U"],
                                       row_status=status)
            return s["U"], status
        U = native.open_foldin(ctx, s["F"], s["row_ptr"], s["col"], s["val"], LAM, case["weighted"],
                               row_status=status)
        return U, status
    if path == "fit":
        U, V = s["U0"].clone(), s["V0"].clone()
        native.open_fit(ctx, s["row_ptr"], s["col"], s["val"], U, V, LAM, case["sweeps"], True)
        return U, V
    if path == "predict":
        m, n = case["m"], s["F"].shape[0]
        status = torch.empty(m, dtype=torch.int32, device=s["F"].device)
        P = torch.empty((m, n), device=s["F"].device) if case["want_p"] else None
        idx, saving = native.open_predict(ctx, s["U"], s["F"], s["cap_cpu"], s["cap_gpu"], s["base"], case["gamma"],
                                          P=P, row_status=status)
        return (idx, saving, status) if P is None else (idx, saving, status, P)
    if path == "surrogate":
        used = torch.empty(case["m"], dtype=torch.uint8, device=s["F"].device)
        rho = torch.empty(case["m"], device=s["F"].device)
        U, _ = s["net"].foldin(s["F"], s["row_ptr"], s["col"], s["val"], case["tau"], LAM, False, used_fallback=used,
                               rho=rho, count=False)
        return U, used, rho
    if path == "surrogate_train":
        s["net"].set_weights(s["w0"])
        hist = s["net"].train(s["row_ptr"], s["col"], s["val"], s["target"], case["batch"], 1e-3, case["epochs"],
                              seed=s["seed"])
        return s["net"].get_weights(), hist
    if path == "ncf":
        m = case["m"]
        loss = torch.empty(m, device=s["S"].device)
        status = torch.empty(m, dtype=torch.int32, device=s["S"].device)
        E = native.open_ncf_foldin(ctx, s["S"], s["params"], s["row_ptr"], s["col"], s["val"], case["steps"], 0.5, 1e-3,
                                   loss_out=loss, row_status=status)
        return E, loss, status
    if path == "ncf_train":
        s["p"].copy_(s["p0"])
        hist = native.open_ncf_train(ctx, s["R"], s["p"], case["group"], 1e-3, case["epochs"], seed=s["seed"])
        return s["p"], hist
    if path == "phase":
        return native.open_phase_detect(ctx, s["power"], 60.0, case["window"])
    return native.open_perf_predict(ctx, s["X"], s["params"])


# ------------------------------------------------------------------------------- work of a pass
def _ridge_flops(c, k):
    """The cheaper of the dual and the primal ridge solve of a row with c observations."""
    dual = c * (c + 1) * k + c ** 3 / 3.0 + 2 * c * c + 2 * c * k
    primal = c * k * (k + 1) + 2 * c * k + k ** 3 / 3.0 + 2 * k * k
    return np.minimum(dual, primal)


def work(case):
    path, m = case["path"], case["m"]
    if path == "phase":  # readings up to the report: half of the trace where there is one (nine in ten)
        return dict(bytes=m * (4.0 * case["length"] * 0.55 + 8), flops=m * case["length"] * 0.55)
    if path == "predictor":
        return dict(bytes=32.0 * m, flops=9216.0 * m)
    n, k = case["n_cpu"] * case["n_gpu"], case.get("k", 0)
    ks, p = _pmf(case, n)
    nnz = m * float((ks * p).sum())
    csr = 8.0 * nnz + 8.0 * m
    if path == "foldin":
        return dict(bytes=csr + 4.0 * k * (m + n) + 4.0 * m, flops=m * float((p * _ridge_flops(ks.astype(float), k)).sum()))
    if path == "fit":
        rows = m * float((p * _ridge_flops(ks.astype(float), k)).sum())
        cols = n * float(_ridge_flops(np.array(nnz / n), k))
        per_sweep = 2 * (8.0 * nnz) + 2 * 4.0 * k * (m + n)
        return dict(bytes=case["sweeps"] * per_sweep, flops=case["sweeps"] * (rows + cols))
    if path == "predict":
        return dict(bytes=4.0 * k * (m + n) + 12.0 * m + (4.0 * m * n if case["want_p"] else 0), flops=2.0 * k * n * m)
    params = HIDDEN * (2.0 * n + 1) + HIDDEN * (HIDDEN + 1) + k * (HIDDEN + 1)
    if path == "surrogate":
        net = 4.0 * HIDDEN * nnz + 2.0 * m * HIDDEN * (HIDDEN + k)
        return dict(bytes=csr + 4.0 * params + 4.0 * k * (m + n) + 5.0 * m, flops=net)
    if path == "surrogate_train":
        steps = case["epochs"] * (m // case["batch"])
        seen = steps * case["batch"]
        fwd = 4.0 * HIDDEN * (nnz / m) + 2.0 * HIDDEN * (HIDDEN + k)
        # rows, entries and targets once, the weights and both moments read and written each step
        return dict(bytes=seen * (8.0 * nnz / m + 8 + 4 * k) + steps * 24.0 * params, flops=3.0 * seen * fwd)
    if path == "ncf":
        per_obs = 2.0 * (32 * 64 + 64 * 64 + 64) + 2.0 * (64 + 64 * 64)
        return dict(bytes=csr + 4.0 * NCF_D * (m + n), flops=case["steps"] * (nnz * per_obs + m * 4.0 * 32 * 64))
    steps = case["epochs"] * (m // case["group"])
    net = NCF_H * (2 * NCF_D + 1) + NCF_H * (NCF_H + 1) + NCF_H + 1
    params = (m + n) * NCF_D + net
    return dict(bytes=steps * (4.0 * case["group"] * n + 24.0 * params),
                flops=steps * case["group"] * n * 3 * 2.0 * (2 * NCF_D * NCF_H + NCF_H * NCF_H + NCF_H))


# ------------------------------------------------------------------------------- float64 values
def _solve_spd(A, b):
    """Batched solve of SPD systems by elimination without pivoting (float64)."""
    M = torch.cat([A, b[:, :, None]], 2)
    for p in range(A.shape[1]):
        row = M[:, p, :] / M[:, p, p:p + 1]
        f = M[:, :, p].clone()
        f[:, p] = 0.0
        M -= f[:, :, None] * row[:, None, :]
        M[:, p, :] = row
    return M[:, :, -1]


def _dense_rows(row_ptr, col, val, n, a, b):
    X = _dense_x(row_ptr, col, val, n, a, b)
    return X[:, :n], X[:, n:]


def _half_sweep(R, W, F, lam, weighted):
    """Ridge rows against F: R the values (zero where unobserved), W the 0/1 mask."""
    k = F.shape[1]
    FF = (F[:, :, None] * F[:, None, :]).reshape(F.shape[0], k * k)
    out = torch.zeros((R.shape[0], k), dtype=torch.float64, device=R.device)
    step = max(1, (1 << 28) // (k * k))
    for a in range(0, R.shape[0], step):
        w, r = W[a:a + step], R[a:a + step]
        cnt = w.sum(1)
        A = (w @ FF).reshape(-1, k, k)
        reg = lam * (cnt if weighted else torch.ones_like(cnt))
        A += torch.diag_embed(torch.where(cnt > 0, reg, 1.0)[:, None].expand(-1, k))
        out[a:a + step] = _solve_spd(A, r @ F)
    return out


def _exact_ridge(row_ptr, col, val, F, lam, weighted):
    m, n = row_ptr.numel() - 1, F.shape[0]
    out, step = [], max(1, (1 << 26) // n)
    for a in range(0, m, step):
        R, W = _dense_rows(row_ptr, col, val, n, a, min(a + step, m))
        out.append(_half_sweep(R, W, F.double(), lam, weighted))
    return torch.cat(out)


def _exact_fit(case, s):
    n, k, m = s["V0"].shape[0], case["k"], case["m"]
    U, V = s["U0"].double(), s["V0"].double()
    R, W = _dense_rows(s["row_ptr"], s["col"], s["val"], n, 0, m)
    for _ in range(case["sweeps"]):
        U = _half_sweep(R, W, V, LAM, True)
        G = torch.zeros((n, k * k), dtype=torch.float64, device=U.device)
        step = max(1, (1 << 28) // (k * k))
        for a in range(0, m, step):
            u = U[a:a + step]
            G += W[a:a + step].T @ (u[:, :, None] * u[:, None, :]).reshape(-1, k * k)
        cnt = W.sum(0)
        A = G.reshape(n, k, k) + torch.diag_embed(torch.where(cnt > 0, LAM * cnt, 1.0)[:, None].expand(-1, k))
        V = _solve_spd(A, R.T @ U)
    return U, V


def _exact_surrogate(case, s, w):
    n, k, m = s["F"].shape[0], case["k"], case["m"]
    W1, b1, W2, b2, W3, b3 = _net_split(torch.from_numpy(w).to(_dev()), n, k)
    F, U, rho = s["F"].double(), [], []
    step = max(1, (1 << 26) // n)
    for a in range(0, m, step):
        b = min(a + step, m)
        X = _dense_x(s["row_ptr"], s["col"], s["val"], n, a, b)
        h = _gelu(X @ _bf16(W1).T + b1.double())
        h = _gelu(h @ _bf16(W2).T + b2.double())
        u = h @ _bf16(W3).T + b3.double()
        R, W = X[:, :n], X[:, n:]
        cnt = W.sum(1)
        res = ((((R - u @ F.T) * W) ** 2).sum(1) / cnt.clamp(min=1)).sqrt()
        ridge = _half_sweep(R, W, F, LAM, False)
        U.append(torch.where((res > case["tau"])[:, None], ridge, u))
        rho.append(res)
    return torch.cat(U), None, torch.cat(rho)


def _mix64(z):
    with np.errstate(over="ignore"):
        z = np.asarray(z, np.uint64) + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def _epoch_order(m, seed, epoch):
    """The seeded row order of an epoch, as the C header defines it."""
    h = 1
    while (1 << (2 * h)) < m:
        h += 1
    mask = np.uint64((1 << h) - 1)
    with np.errstate(over="ignore"):
        keys = [_mix64(_mix64(np.uint64(seed)) + np.uint64(4 * epoch + r)) for r in range(4)]
    x = np.arange(m, dtype=np.uint64)
    todo = np.ones(m, bool)
    while todo.any():
        L, R = x[todo] >> np.uint64(h), x[todo] & mask
        for key in keys:
            L, R = R, L ^ (_mix64(R ^ key) & mask)
        x[todo] = (L << np.uint64(h)) | R
        todo &= x >= np.uint64(m)
    return x.astype(np.int64)


class _Adam:
    def __init__(self, w):
        self.w, self.m, self.v, self.t = w, torch.zeros_like(w), torch.zeros_like(w), 0

    def step(self, g, lr):
        self.t += 1
        self.m = 0.9 * self.m + 0.1 * g
        self.v = 0.999 * self.v + 0.001 * g * g
        self.w = self.w - lr * (self.m / (1 - 0.9 ** self.t)) / ((self.v / (1 - 0.999 ** self.t)).sqrt() + 1e-8)


def _gelu_grad(z):
    return 0.5 * (1.0 + torch.erf(z / math.sqrt(2.0))) + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)


def _exact_surrogate_train(case, s):
    n, k, m, B = s["F"].shape[0], case["k"], case["m"], case["batch"]
    opt = _Adam(torch.from_numpy(s["w0"]).to(_dev()).double())
    target, hist = s["target"].double(), []
    X = _dense_x(s["row_ptr"], s["col"], s["val"], n, 0, m)
    for e in range(case["epochs"]):
        order = torch.from_numpy(_epoch_order(m, s["seed"], e)).to(_dev())
        losses = []
        for b in range(m // B):
            rows = order[b * B:(b + 1) * B]
            W1, b1, W2, b2, W3, b3 = _net_split(opt.w, n, k)
            W1, W2, W3 = _bf16(W1), _bf16(W2), _bf16(W3)
            x = X[rows]
            z1 = x @ W1.T + b1
            h1 = _gelu(z1)
            z2 = h1 @ W2.T + b2
            h2 = _gelu(z2)
            d = h2 @ W3.T + b3 - target[rows]
            losses.append((d * d).mean())
            d = 2.0 * d / d.numel()
            d2 = (d @ W3) * _gelu_grad(z2)
            d1 = (d2 @ W2) * _gelu_grad(z1)
            opt.step(torch.cat([(d1.T @ x).ravel(), d1.sum(0), (d2.T @ h1).ravel(), d2.sum(0), (d.T @ h2).ravel(),
                                d.sum(0)]), 1e-3)
        hist.append(torch.stack(losses).mean())
    return opt.w.cpu().numpy(), torch.stack(hist).cpu().numpy()


SELU_A, SELU_L = 1.6732632423543772, 1.0507009873554805


def _selu(z):
    e = torch.exp(z.clamp(max=0.0))
    pos = z > 0
    return torch.where(pos, SELU_L * z, SELU_L * SELU_A * (e - 1.0)), torch.where(pos, SELU_L, SELU_L * SELU_A * e)


def _exact_ncf(case, s):
    m, n = case["m"], s["S"].shape[0]
    p = {k: v.double() for k, v in s["params"].items()}
    W1e, W2 = p["W1"][:, :NCF_D], p["W2"]
    C = s["S"].double() @ p["W1"][:, NCF_D:].T + p["b1"]
    E, loss = [], []
    for a in range(0, m, 16384):
        b = min(a + 16384, m)
        e0, e1 = int(s["row_ptr"][a]), int(s["row_ptr"][b])
        cnt = s["row_ptr"][a + 1:b + 1] - s["row_ptr"][a:b]
        rows = torch.repeat_interleave(torch.arange(b - a, device=_dev()), cnt, output_size=e1 - e0)
        r = s["val"][e0:e1].double()
        c = C[s["col"][e0:e1].long()]
        q = cnt.double().clamp(min=1)
        e = torch.zeros((b - a, NCF_D), dtype=torch.float64, device=_dev())
        for it in range(case["steps"] + 1):
            h1, g1 = _selu((e @ W1e.T)[rows] + c)
            h2, g2 = _selu(h1 @ W2.T + p["b2"])
            res = h2 @ p["w3"] + p["b3"] - r
            if it == case["steps"]:
                sq = torch.zeros(b - a, dtype=torch.float64, device=_dev()).index_add_(0, rows, res * res)
                loss.append(sq / q + 1e-3 * (e * e).sum(1))
                break
            dz1 = (((2.0 * res / q[rows])[:, None] * p["w3"] * g2) @ W2) * g1
            g = torch.zeros((b - a, NCF_H), dtype=torch.float64, device=_dev()).index_add_(0, rows, dz1)
            e = e - 0.5 * (g @ W1e + 2e-3 * e)
        E.append(e)
    return torch.cat(E), torch.cat(loss), None


def _exact_ncf_train(case, s):
    m, n, G = case["m"], s["R"].shape[1], case["group"]
    opt, R, hist = _Adam(s["p0"].double()), s["R"].double(), []
    for ep in range(case["epochs"]):
        order = torch.from_numpy(_epoch_order(m, s["seed"], ep)).to(_dev())
        losses = []
        for b in range(m // G):
            apps = order[b * G:(b + 1) * G]
            E, S, net = native.ncf_unpack(opt.w, m, n)
            X = torch.cat([E[apps].repeat_interleave(n, 0), S.repeat(G, 1)], 1)
            h1, g1 = _selu(X @ net["W1"].T + net["b1"])
            h2, g2 = _selu(h1 @ net["W2"].T + net["b2"])
            d = h2 @ net["w3"] + net["b3"] - R[apps].reshape(-1)
            losses.append((d * d).mean())
            d = 2.0 * d / d.numel()
            d2 = d[:, None] * net["w3"] * g2
            d1 = (d2 @ net["W2"]) * g1
            dX = (d1 @ net["W1"]).reshape(G, n, 2 * NCF_D)
            gE = torch.zeros_like(E)
            gE[apps] = dX[:, :, :NCF_D].sum(1)
            opt.step(torch.cat([gE.ravel(), dX[:, :, NCF_D:].sum(0).ravel(), (d1.T @ X).ravel(), d1.sum(0),
                                (d2.T @ h1).ravel(), d2.sum(0), h2.T @ d, d.sum()[None]]), 1e-3)
        hist.append(torch.stack(losses).mean())
    return opt.w, torch.stack(hist).cpu().numpy()


def _exact_predict(case, s):
    U, V = s["U"].double(), s["F"].double()
    w = s["cap_cpu"].double() + s["cap_gpu"].double()
    saving, P = [], []
    step = max(1, (1 << 27) // V.shape[0])
    for a in range(0, case["m"], step):
        p = U[a:a + step] @ V.T
        pb = p[:, s["base"]:s["base"] + 1]
        E = torch.where((p > 0) & (1.0 - p / pb <= case["gamma"]), w / p, math.inf)
        best = (w[s["base"]] - E.min(1).values) / w[s["base"]]
        saving.append(torch.where(pb[:, 0] > 0, best, 0.0))
        if case["want_p"]:
            P.append(p)
    out = (None, torch.cat(saving), None)
    return out + (torch.cat(P),) if case["want_p"] else out


def _exact_predictor(s):
    p = {k: v.double() for k, v in s["params"].items()}
    out = []
    for x in s["X"].split(1 << 20):
        h = ((x.double() - p["mu"]) * p["rs"]) @ _bf16(p["W1"]).T + p["b1"]
        h = h.clamp(min=0) @ _bf16(p["W2"]).T + p["b2"]
        out.append(h.clamp(min=0) @ p["w3"] + p["b3"])
    return torch.cat(out)


def exact(case, seed):
    path = case["path"]
    s = prepare(case, seed)
    if path == "foldin":
        return _exact_ridge(s["row_ptr"], s["col"], s["val"], s["F"], LAM, case["weighted"]), None
    if path == "fit":
        return _exact_fit(case, s)
    if path == "predict":
        return _exact_predict(case, s)
    if path == "surrogate":
        return _exact_surrogate(case, s, _surrogate_weights(case["n_cpu"], case["n_gpu"], case["k"]))
    if path == "surrogate_train":
        return _exact_surrogate_train(case, s)
    if path == "ncf":
        return _exact_ncf(case, s)
    if path == "ncf_train":
        return _exact_ncf_train(case, s)
    if path == "predictor":
        return _exact_predictor(s)
    return None
