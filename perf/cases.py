"""The work that users of this package have it do, as cases that can be timed.

Every case goes through the public entry points of ``paper_1705_04159_amd``:

* ``sweeps``  -- Gibbs sweeps of Algorithm 1 driven call by call
  (``sample_hyper``, ``update_side`` for both sides, ``predict_test``), then
  the factors read back (training, with the RMSE watched);
* ``steps``   -- one such sweep with the state read back after every call (a
  program that exchanges or checks the state between the steps);
* ``update``  -- one side's conditional update and its new factor;
* ``hyper``   -- one hyperparameter draw;
* ``predict`` -- predictions for given (user, movie) pairs.

The rating matrices have the shapes of the workloads in ``synth`` (planted
values, skewed degrees) and are made on the GPU from the seed.
"""
import math

import numpy as np
import torch

import paper_1705_04159_amd as bp

ALPHA, BETA0 = 2.0, 2.0
EXACT_WORK = 3e10  # FLOP beyond which the 64-bit reference would take too long


def listed():
    return [
        # the plain planted problem, FP64 throughout: every launch is tiny, a sweep is latency
        {"name": "sweeps-planted-fp64", "kind": "sweeps", "shape": "planted", "M": 1000, "N": 500,
         "nnz": 20000, "K": 10, "prec": "fp64", "n": 20, "reorder": False},
        # FP64 at a rank used in earnest (reference runs of a mid-sized recommender)
        {"name": "sweeps-fp64-k32", "kind": "sweeps", "shape": "ratings", "M": 6000, "N": 3500,
         "nnz": 500000, "K": 32, "prec": "fp64", "n": 5, "reorder": False},
        # the 20M-rating recommender at full size: the benchmark's default workload
        {"name": "sweeps-20m-k32", "kind": "sweeps", "shape": "ratings", "M": 138493, "N": 26744,
         "nnz": 20000263, "K": 32, "prec": "fp32", "n": 20, "reorder": True},
        # an eighth of the users of the 100M-rating recommender, all of its movies
        {"name": "sweeps-100m-k100", "kind": "sweeps", "shape": "zipf", "M": 60024, "N": 17770,
         "nnz": 12560063, "K": 100, "prec": "fp32", "n": 10, "reorder": True},
        # the same matrix in the BF16-Gram form, movie side alone (the gather-bound side)
        {"name": "update-100m-bf16", "kind": "update", "shape": "zipf", "M": 60024, "N": 17770,
         "nnz": 12560063, "K": 100, "prec": "bf16", "side": "V", "reorder": True},
        # compound x protein activities (a quarter of the compounds): rows with a handful of ratings
        {"name": "sweeps-compound-k64", "kind": "sweeps", "shape": "compound", "M": 120875,
         "N": 5775, "nnz": 500000, "K": 64, "prec": "fp32", "n": 50, "reorder": False},
        # a small problem of odd sizes driven call by call: launches, synchronisations, read-backs
        {"name": "steps-small-k33", "kind": "steps", "shape": "ratings", "M": 2011, "N": 997,
         "nnz": 100003, "K": 33, "prec": "fp32", "reorder": False},
        # users of a mid-sized recommender against a fixed V, FP32, K = 16
        {"name": "update-users-k16", "kind": "update", "shape": "ratings", "M": 20000, "N": 4001,
         "nnz": 2000000, "K": 16, "prec": "fp32", "side": "U", "reorder": False},
        # the hyperparameter draw at a large rank
        {"name": "hyper-k100", "kind": "hyper", "shape": "ratings", "M": 120047, "N": 1000,
         "nnz": 1000000, "K": 100, "prec": "fp32", "side": "U", "reorder": False},
        # scores for a list of pairs (a ranking service's re-scoring call)
        {"name": "predict-20k", "kind": "predict", "shape": "ratings", "M": 50000, "N": 20000,
         "nnz": 1000000, "K": 32, "prec": "fp32", "pairs": 20000, "reorder": True},
        # the largest rank, with more ratings a row than a wave's worth of them
        {"name": "update-movies-k128", "kind": "update", "shape": "ratings", "M": 30011, "N": 8000,
         "nnz": 3000000, "K": 128, "prec": "fp32", "side": "V", "reorder": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sweeps", "sweeps", "sweeps", "steps", "update", "update", "hyper", "predict"])
    shape = rng.choice(["ratings", "zipf", "compound"])
    prec = rng.choice(["fp32", "fp32", "fp32", "fp64"] + (["bf16"] if kind in ("update", "hyper") else []))
    K = rng.randint(5, 64) if prec == "fp64" else rng.randint(8, 128)
    if kind == "hyper":
        return {"kind": kind, "shape": "ratings", "M": _log_int(rng, 2000, 200000), "N": 500,
                "nnz": 50000, "K": K, "prec": prec, "side": "U", "reorder": False}
    hi = 500000 if prec == "fp64" else 4000000
    if kind == "steps":
        hi = 500000
    nnz = _log_int(rng, 20000, hi)
    if shape == "compound":
        M, N = nnz // rng.randint(4, 10), max(300, nnz // rng.randint(300, 500))
    else:
        M, N = nnz // rng.randint(40, 200), max(200, nnz // rng.randint(200, 900))
    N = max(N, 12 * nnz // M)  # sparse
    c = {"kind": kind, "shape": shape, "M": M, "N": N, "nnz": nnz, "K": K, "prec": prec,
         "reorder": rng.random() < 0.5}
    if kind == "sweeps":
        c["n"] = rng.randint(1, 5) if prec == "fp64" else rng.randint(2, 12)
    elif kind == "update":
        c["side"] = rng.choice(["U", "V"])
    elif kind == "predict":
        c["pairs"] = _log_int(rng, 100, 200000)
    return c


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------
def _mandelbrot(n, q, s, gen, dev):
    w = (torch.arange(n, device=dev, dtype=torch.float64) + 1.0 + q) ** (-s)
    return w[torch.randperm(n, generator=gen, device=dev)]


def _weights(case, gen, dev):
    """Popularity of the users and movies of a shape."""
    M, N, shape = case["M"], case["N"], case["shape"]
    if shape == "planted":
        return _mandelbrot(M, 0, 1.2, gen, dev), _mandelbrot(N, 0, 1.2, gen, dev)
    if shape == "zipf":
        return _mandelbrot(M, M / 400, 1.1, gen, dev), _mandelbrot(N, N / 170, 1.1, gen, dev)
    if shape == "compound":
        heavy = 0.85 ** torch.arange(20, device=dev, dtype=torch.float64)
        light = torch.exp(1.9 * torch.randn(N - 20, generator=gen, device=dev, dtype=torch.float64))
        wm = torch.cat([0.3 * heavy / heavy.sum(), 0.7 * light / light.sum()])
        return _mandelbrot(M, 50, 1.0, gen, dev), wm[torch.randperm(N, generator=gen, device=dev)]
    u = torch.rand(M, generator=gen, device=dev, dtype=torch.float64)
    return torch.clamp(20.0 * (1.0 - u) ** (-1.0), max=9254.0), _mandelbrot(N, N / 500, 1.0, gen, dev)


class _Ratings:
    """Training ratings as CSR and held-out triples, on the host."""


def _ratings(case, gen, dev):
    """nnz distinct (user, movie) pairs with the shape's degrees, planted values
    with noise; a tenth is held out.  Also the planted factors (float32)."""
    M, N, K, nnz = case["M"], case["N"], case["K"], case["nnz"]
    wu, wm = _weights(case, gen, dev)
    cu, cm = torch.cumsum(wu / wu.sum(), 0), torch.cumsum(wm / wm.sum(), 0)
    key = torch.zeros(0, dtype=torch.int64, device=dev)
    for _ in range(30):
        n = int(1.15 * (nnz - key.numel())) + 64
        r = torch.searchsorted(cu, torch.rand(n, generator=gen, device=dev, dtype=torch.float64))
        c = torch.searchsorted(cm, torch.rand(n, generator=gen, device=dev, dtype=torch.float64))
        key = torch.unique(torch.cat([key, r.clamp_(max=M - 1) * N + c.clamp_(max=N - 1)]))
        if key.numel() >= nnz:
            break
    if key.numel() < nnz:
        raise ValueError("could not place %d distinct pairs" % nnz)
    keep = torch.zeros(key.numel(), dtype=torch.bool, device=dev)
    keep[torch.randperm(key.numel(), generator=gen, device=dev)[:nnz]] = True
    key = key[keep]
    rows, cols = key // N, key % N
    sd = K ** -0.25
    Us = torch.randn(M, K, generator=gen, device=dev) * sd
    Vs = torch.randn(N, K, generator=gen, device=dev) * sd
    val = 0.5 * torch.randn(nnz, generator=gen, device=dev)
    for s in range(0, nnz, 1 << 22):
        e = slice(s, min(nnz, s + (1 << 22)))
        val[e] += 3.5 + (Us[rows[e]] * Vs[cols[e]]).sum(1)
    if case["shape"] == "ratings":  # half stars
        val = (torch.round(val * 2.0) / 2.0).clamp(0.5, 5.0)
    elif case["shape"] == "zipf":  # whole stars
        val = torch.round(val).clamp(1.0, 5.0)
    test = torch.rand(nnz, generator=gen, device=dev) < 0.1
    r = _Ratings()
    r.M, r.N = M, N
    tr = ~test
    r.csr_ptr = np.zeros(M + 1, np.int64)
    np.cumsum(torch.bincount(rows[tr], minlength=M).cpu().numpy(), out=r.csr_ptr[1:])
    r.csr_col = cols[tr].to(torch.int32).cpu().numpy()
    r.csr_val = val[tr].cpu().numpy()
    r.test_row = rows[test].to(torch.int32).cpu().numpy()
    r.test_col = cols[test].to(torch.int32).cpu().numpy()
    r.test_val = val[test].cpu().numpy()
    return r, Us, Vs


def _prior(K, rng):
    """A mean and a precision of the size that the hyper draws have."""
    A = rng.standard_normal((K, 2 * K))
    return 0.1 * rng.standard_normal(K), math.sqrt(K) * (0.7 * np.eye(K) + 0.3 * (A @ A.T) / (2 * K))


def _inputs(case, seed):
    """Everything the seed decides, on the host (factors also where given)."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    rng = np.random.default_rng(int(seed))
    x = {"seed": int(seed) * 2 + 1}
    x["ratings"], Us, Vs = _ratings(case, gen, dev)
    if case["kind"] in ("update", "hyper", "predict"):
        f = np.float64 if case["prec"] == "fp64" else np.float32
        x["U"], x["V"] = Us.cpu().numpy().astype(f), Vs.cpu().numpy().astype(f)
        x["hyper"] = _prior(case["K"], rng)
    if case["kind"] == "predict":
        x["rows"] = rng.integers(0, case["M"], case["pairs"]).astype(np.int32)
        x["cols"] = rng.integers(0, case["N"], case["pairs"]).astype(np.int32)
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    kind = case["kind"]
    s = bp.Sampler(x["ratings"], case["K"], prec=case["prec"], alpha=ALPHA, beta0=BETA0, seed=x["seed"],
                   reorder=case["reorder"])
    state = {"case": case, "s": s, "t": 1}
    if kind in ("update", "hyper", "predict"):
        s.set_factor(bp.SIDE_U, x["U"])
        s.set_factor(bp.SIDE_V, x["V"])
        for side in (bp.SIDE_U, bp.SIDE_V):
            s.set_hyper(side, *x["hyper"])
    if kind == "predict":
        state["rows"], state["cols"] = x["rows"], x["cols"]
    return state


def run(state):
    case, s = state["case"], state["s"]
    kind = case["kind"]
    if kind == "predict":
        return {"out": s.predict(state["rows"], state["cols"])}
    t = state["t"]
    if kind == "sweeps":
        rmse = []
        for t in range(t, t + case["n"]):
            for side in (bp.SIDE_V, bp.SIDE_U):
                s.sample_hyper(side, t)
                s.update_side(side, t)
            rmse.append(s.predict_test(t))
        state["t"] = t + 1
        return {"rmse": _as(case, np.array(rmse)), "U": s.get_factor(bp.SIDE_U), "V": s.get_factor(bp.SIDE_V)}
    state["t"] += 1
    if kind == "hyper":
        side = bp.SIDE_U if case["side"] == "U" else bp.SIDE_V
        s.sample_hyper(side, t)
        mu, Lam = s.get_hyper(side)
        return {"mu": mu, "Lam": Lam}
    if kind == "update":
        side = bp.SIDE_U if case["side"] == "U" else bp.SIDE_V
        s.update_side(side, t)
        return {"X": s.get_factor(side)}
    out = {}
    for name, side in (("V", bp.SIDE_V), ("U", bp.SIDE_U)):
        s.sample_hyper(side, t)
        mu, Lam = s.get_hyper(side)
        s.update_side(side, t)
        out[name] = s.get_factor(side)
        out["mu" + name], out["Lam" + name] = _as(case, mu), _as(case, Lam)
    avg, last = s.predict_test(t)
    out["rmse"] = _as(case, np.array([avg, last]))
    return out


def _as(case, x):
    """Quantities that follow from FP32 factors, at the precision that they have."""
    return x if case["prec"] == "fp64" else np.asarray(x, np.float32)


def _gram_flops(case, sides=2):
    K = case["K"]
    return sides * 0.9 * case["nnz"] * (K * (K + 1) + 2.0 * K)


def _row_flops(K):
    return K ** 3 / 3.0 + 2.0 * K * K


def work(case):
    kind, K = case["kind"], case["K"]
    es = 8 if case["prec"] == "fp64" else 4
    M, N, nnz = case["M"], case["N"], 0.9 * case["nnz"]
    if kind == "predict":
        n = case["pairs"]
        return {"bytes": n * 12.0 + es * K * (min(n, M) + min(n, N)), "flops": 2.0 * n * K}
    if kind == "hyper":
        return {"bytes": float(es * M * K + 8 * K * K),
                "flops": M * K * (K + 1.0) + 4.0 * K ** 3}
    if kind == "update":
        rows = M if case["side"] == "U" else N
        return {"bytes": (4.0 + es) * nnz + es * K * (M + N),
                "flops": _gram_flops(case, 1) + rows * _row_flops(K)}
    n = case.get("n", 1)
    per_bytes = 2 * (4.0 + es) * nnz + 2.0 * es * K * (M + N) + 0.1 * case["nnz"] * 20.0
    per_flops = _gram_flops(case) + (M + N) * (_row_flops(K) + K * (K + 1.0))
    return {"bytes": n * per_bytes, "flops": n * per_flops}


# --------------------------------------------------------------------------
# The same in 64 bits (numpy), from the definitions of the model and its noise
# --------------------------------------------------------------------------
def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on arrays of counters (broadcast), four uint64 words < 2^32."""
    m = np.uint64(0xFFFFFFFF)
    c = [np.asarray(v, np.uint64) for v in (c0, c1, c2, c3)]
    c = list(np.broadcast_arrays(*c))
    k0, k1 = int(seed) & 0xFFFFFFFF, int(seed) >> 32
    sh = np.uint64(32)
    for _ in range(10):
        a = np.uint64(0xD2511F53) * c[0]
        b = np.uint64(0xCD9E8D57) * c[2]
        c = [(b >> sh) ^ c[1] ^ np.uint64(k0), b & m, (a >> sh) ^ c[3] ^ np.uint64(k1), a & m]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _unit(w):
    return (w.astype(np.float64) + 0.5) * 2.0 ** -32


def _normals(n, c0, c1, stream, sub, c3, seed):
    """Normals 0..n-1 of each (c0, c1, c3); c0 may be an array: shape (len(c0), n)."""
    blk = np.arange((n + 3) // 4, dtype=np.uint64)[None, :] + np.uint64(sub)
    w = _philox(np.atleast_1d(np.asarray(c0, np.uint64))[:, None], c1, np.uint64(stream << 24) | blk, c3, seed)
    z = _box(w)
    return np.stack(z, -1).reshape(z[0].shape[0], -1)[:, :n]


def _box(w):
    ra, rb = np.sqrt(-2.0 * np.log(_unit(w[0]))), np.sqrt(-2.0 * np.log(_unit(w[2])))
    ta, tb = 2.0 * np.pi * _unit(w[1]), 2.0 * np.pi * _unit(w[3])
    return ra * np.cos(ta), ra * np.sin(ta), rb * np.cos(tb), rb * np.sin(tb)


def _chi2(dof, k, t, stream, seed):
    d = 0.5 * dof - 1.0 / 3.0
    c = 1.0 / math.sqrt(9.0 * d)
    for attempt in range(4096):
        w = _philox(k, t, stream << 24, attempt, seed)
        x = float(_box(w)[0])
        v = (1.0 + c * x) ** 3
        if v > 0 and math.log(float(_unit(w[2]))) < 0.5 * x * x + d - d * v + d * math.log(v):
            return 2.0 * d * v
    raise ValueError("no chi-square draw")


def _hyper_exact(X, seed, t, stream):
    """Normal-Wishart posterior draw with mu0 = 0, beta0 = 2, nu0 = K, W0 = I."""
    n, K = X.shape
    xbar = X.mean(0)
    S = (X - xbar).T @ (X - xbar)
    Winv = np.eye(K) + S + BETA0 * n / (BETA0 + n) * np.outer(xbar, xbar)
    LW = np.linalg.cholesky(np.linalg.inv(Winv))
    A = np.zeros((K, K))
    A[np.tril_indices(K, -1)] = _normals_seq(K * (K - 1) // 2, t, stream, 1, seed)
    for k in range(K):
        A[k, k] = math.sqrt(_chi2(K + n - k, k, t, stream, seed))
    B = LW @ A
    z = _normals_seq(K, t, stream, 2, seed)
    return n * xbar / (BETA0 + n) + np.linalg.solve(B.T, z) / math.sqrt(BETA0 + n), B @ B.T


def _normals_seq(n, t, stream, sub, seed):
    """Normals of counters (block, t, stream << 24 | sub, 0), block by block."""
    w = _philox(np.arange((n + 3) // 4, dtype=np.uint64), t, (stream << 24) | sub, 0, seed)
    return np.stack(_box(w), -1).reshape(-1)[:n]


def _rows_exact(ptr, idx, rc, Y, mu, Lam, noise_row, t, stream, seed):
    """Every row's conditional draw x = L^-T (L^-1 b + z)."""
    rows, K = len(ptr) - 1, Y.shape[1]
    out = np.empty((rows, K))
    Lmu = Lam @ mu
    for s in range(0, rows, 4096):
        e = min(rows, s + 4096)
        P = np.empty((e - s, K, K))
        b = np.empty((e - s, K))
        for i in range(s, e):
            y = Y[idx[ptr[i]:ptr[i + 1]]]
            P[i - s] = Lam + ALPHA * (y.T @ y)
            b[i - s] = Lmu + ALPHA * (rc[ptr[i]:ptr[i + 1]] @ y)
        L = np.linalg.cholesky(P)
        w = np.linalg.solve(L, b[..., None])[..., 0]
        w += _normals(K, noise_row[s:e], t, stream, 0, 0, seed)
        out[s:e] = np.linalg.solve(np.swapaxes(L, 1, 2), w[..., None])[..., 0]
    return out


class _Chain:
    """The sampler of Algorithm 1 in numpy, in the caller's ids."""

    def __init__(self, r, K, seed, reorder):
        self.r, self.K, self.seed = r, K, seed
        M, N = r.M, r.N
        self.rbar = r.csr_val.astype(np.float64).mean()
        rows = np.repeat(np.arange(M), np.diff(r.csr_ptr))
        o = np.argsort(r.csr_col, kind="stable")
        cptr = np.concatenate([[0], np.cumsum(np.bincount(r.csr_col, minlength=N))])
        rc = r.csr_val.astype(np.float64) - self.rbar
        self.csr = (r.csr_ptr, r.csr_col, rc)
        self.csc = (cptr, rows[o], rc[o])
        self.noise = [np.arange(M), np.arange(N)]
        if reorder:  # the noise counters follow the degree order
            for q, deg in enumerate((np.diff(r.csr_ptr), np.diff(cptr))):
                self.noise[q] = np.empty(len(deg), np.int64)
                self.noise[q][np.argsort(-deg, kind="stable")] = np.arange(len(deg))
        self.pred, self.n = np.zeros(len(r.test_row)), 0

    def init(self, f):
        sc = self.K ** -0.25
        self.X = [(sc * _normals(self.K, nz, 0, st, 0, 0, self.seed)).astype(f).astype(np.float64)
                  for nz, st in zip(self.noise, (5, 6))]

    def hyper(self, side, t):
        return _hyper_exact(self.X[side], self.seed, t, 3 + side)

    def update(self, side, t, mu, Lam):
        self.X[side] = _rows_exact(*(self.csr, self.csc)[side], self.X[1 - side], mu, Lam, self.noise[side],
                                   t, 1 + side, self.seed)

    def predict(self):
        p = (self.X[0][self.r.test_row] * self.X[1][self.r.test_col]).sum(1) + self.rbar
        self.pred += p
        self.n += 1
        v = self.r.test_val.astype(np.float64)
        return [math.sqrt(((q - v) ** 2).mean()) for q in (self.pred / self.n, p)]


def exact(case, seed):
    kind = case["kind"]
    if work(case)["flops"] > EXACT_WORK or (case["M"] > 60000 and kind != "hyper"):
        return None
    x = _inputs(case, seed)
    c = _Chain(x["ratings"], case["K"], x["seed"], case["reorder"])
    f = np.float64 if case["prec"] == "fp64" else np.float32
    if "U" in x:
        c.X = [x["U"].astype(np.float64), x["V"].astype(np.float64)]
    else:
        c.init(f)
    if kind == "predict":
        return {"out": (c.X[0][x["rows"]] * c.X[1][x["cols"]]).sum(1) + c.rbar}
    side = 0 if case.get("side") == "U" else 1
    if kind == "hyper":
        mu, Lam = c.hyper(side, 1)
        return {"mu": mu, "Lam": Lam}
    if kind == "update":
        if case["prec"] == "bf16":  # the gathered rows are rounded to BF16 by definition
            y = torch.from_numpy(c.X[1 - side]).to(torch.float32).to(torch.bfloat16).to(torch.float64)
            c.X[1 - side] = y.numpy()
        c.update(side, 1, *x["hyper"])
        return {"X": c.X[side]}
    n = case.get("n", 1)
    rm, out = [], {}
    for t in range(1, n + 1):
        for name, sd in (("V", 1), ("U", 0)):
            mu, Lam = c.hyper(sd, t)
            c.update(sd, t, mu, Lam)
            out["mu" + name], out["Lam" + name] = mu, Lam
        rm.append(c.predict())
    rm = np.array(rm)
    if kind == "sweeps":
        return {"rmse": rm, "U": c.X[0], "V": c.X[1]}
    return dict(out, U=c.X[0], V=c.X[1], rmse=rm[0])
