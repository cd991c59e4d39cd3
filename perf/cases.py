"""Cases for timing the library through its public entry points.

Every case is one call a user's program makes (a solve, a colouring, a
regularisation path, an FP64 check, a batch of server requests) on a seeded
synthetic problem of the sizes that the repository's own workloads and tests
use: Bernoulli matrices (dense-ish small problems, serving requests, the
binary path) and Zipf ones (text-like, a few columns holding most entries).

`listed()` names the cases, `draw()` gives others of the same ranges,
`prepare()` makes the inputs on the GPU, `run()` is the timed call, `work()`
what it cannot do without and `exact()` the same result in 64-bit torch.
"""
import math

import torch

from paper_1206_6409_amd import gencd as G

_GOLD = 0x9E3779B97F4A7C15
_M64 = (1 << 64) - 1


def _dev():
    return "cuda" if torch.cuda.is_available() else "cpu"


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _gen(seed, dev):
    return torch.Generator(device=dev).manual_seed(int(seed))


def _segsum(v, ptr):
    """Sums of the consecutive runs [ptr[i], ptr[i + 1])."""
    acc = torch.cat([torch.zeros(1, dtype=v.dtype, device=v.device), torch.cumsum(v, 0)])
    return acc[ptr[1:]] - acc[ptr[:-1]]


def _csc(n, k, cols, rows, vals):
    """CSC arrays from entries already sorted by (column, row)."""
    col_ptr = torch.searchsorted(cols, torch.arange(k + 1, device=cols.device))
    return col_ptr, rows.to(torch.int32), vals.to(torch.float32)


def _bernoulli(n, k, density, binary, g, dev):
    """Entries present independently: the gaps between the nonzero cells (in
    column-major order) are geometric."""
    cells = n * k
    mean = cells * density
    m = int(mean + 8.0 * math.sqrt(mean) + 16)
    u = torch.rand(m, generator=g, device=dev, dtype=torch.float64).clamp_(min=1e-300)
    pos = torch.cumsum((torch.log(u) / math.log1p(-density)).to(torch.int64) + 1, 0) - 1
    pos = pos[pos < cells]
    cols = torch.div(pos, n, rounding_mode="floor")
    rows = pos - cols * n
    vals = torch.ones(pos.numel(), device=dev) if binary else \
        torch.randn(pos.numel(), generator=g, device=dev)
    return _csc(n, k, cols, rows, vals)


def _zipf(n, k, a, mean_len, lognormal, g, dev):
    """Rows of 1 + Poisson(mean - 1) distinct column ranks from Zipf(a),
    ranks mapped to columns at random; lognormal values are scaled to rows of
    unit length, others are N(0, 1)."""
    lens = 1 + torch.poisson(torch.full((n,), float(mean_len - 1), device=dev), generator=g)
    left = lens.to(torch.int64).clamp_(max=k)
    cdf = torch.cumsum(torch.arange(1, k + 1, device=dev, dtype=torch.float64) ** (-a), 0)
    cdf /= cdf[-1].clone()
    have = torch.zeros(0, dtype=torch.int64, device=dev)
    ids = torch.arange(n, device=dev)
    for _ in range(200):
        r = torch.repeat_interleave(ids, left)
        if r.numel() == 0:
            break
        u = torch.rand(r.numel(), generator=g, device=dev, dtype=torch.float64)
        new = torch.unique(r * k + torch.searchsorted(cdf, u).clamp_(max=k - 1))
        if have.numel():
            at = torch.searchsorted(have, new).clamp_(max=have.numel() - 1)
            new = new[have[at] != new]
        left = left - torch.bincount(torch.div(new, k, rounding_mode="floor"), minlength=n)
        have = torch.sort(torch.cat([have, new]))[0]
    rows = torch.div(have, k, rounding_mode="floor")
    cols = torch.randperm(k, generator=g, device=dev)[have - rows * k]
    vals = torch.randn(have.numel(), generator=g, device=dev, dtype=torch.float64)
    if lognormal:
        vals = vals.exp()
        ptr = torch.zeros(n + 1, dtype=torch.int64, device=dev)
        torch.cumsum(torch.bincount(rows, minlength=n), 0, out=ptr[1:])
        vals = vals / _segsum(vals * vals, ptr).clamp_(min=1e-30).sqrt()[rows]
    order = torch.argsort(cols * n + rows)
    return _csc(n, k, cols[order], rows[order], vals[order])


def _problem(case, seed):
    """Matrix, labels and lambda of a case, from the seed alone."""
    dev = _dev()
    g = _gen(seed, dev)
    n, k = case["n"], case["k"]
    if case["matrix"] == "zipf":
        col_ptr, rows, val = _zipf(n, k, case["a"], case["mean_len"], case["loss"] == G.LOGISTIC,
                                   g, dev)
    else:
        col_ptr, rows, val = _bernoulli(n, k, case["density"], case.get("binary", False), g, dev)
    lens = col_ptr[1:] - col_ptr[:-1]
    cid = torch.repeat_interleave(torch.arange(k, device=dev), lens)
    # labels from a sparse ground truth on non-empty columns
    live = torch.nonzero(lens).reshape(-1)
    wt = torch.zeros(k, dtype=torch.float64, device=dev)
    sup = live[torch.randperm(live.numel(), generator=g, device=dev)[:case["support"]]]
    wt[sup] = torch.randn(sup.numel(), generator=g, device=dev, dtype=torch.float64)
    v64 = val.double()
    z = torch.zeros(n, dtype=torch.float64, device=dev).index_add_(0, rows.long(), v64 * wt[cid])
    if case["loss"] == G.LOGISTIC:
        u = torch.rand(n, generator=g, device=dev, dtype=torch.float64)
        y = torch.where(u < torch.sigmoid(z), 1.0, -1.0).float()
        r = -0.5 * y.double()
    else:
        y = (z + 0.1 * torch.randn(n, generator=g, device=dev, dtype=torch.float64)).float()
        r = -y.double()
    grad = _segsum(v64 * r[rows.long()], col_ptr)
    lmax = float(grad.abs().max()) / n
    return {"n": n, "k": k, "col_ptr": col_ptr, "row_idx": rows, "val": val, "y": y,
            "lmax": lmax, "lam": case.get("lam_ratio", 1.0) * lmax}


def _requests(case, seed):
    """The request cases of a server batch: sizes, densities and lambdas of
    the serving stream's law (its lower size range)."""
    g = torch.Generator().manual_seed(int(case["mix"]))
    out = []
    for i in range(case["requests"]):
        u = torch.rand(5, generator=g).tolist()
        lo, hi = case["ratio_lo"], 0.5
        out.append({"matrix": "bernoulli", "n": int(1000 + u[0] * (case["n"] - 1000)),
                    "k": int(1000 + u[1] * (case["k"] - 1000)),
                    "density": 0.001 + 0.019 * u[2], "support": 50,
                    "loss": G.LOGISTIC if u[3] < 0.5 else G.SQUARED,
                    "lam_ratio": lo * (hi / lo) ** u[4], "rule": "shotgun", "select": 0,
                    "block": 1, "tol": 1e-6, "max_epochs": case["max_epochs"], "check_every": 0})
    return out, [seed * 64 + i for i in range(case["requests"])]


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def _zipf_case(n, k, a=1.1, mean_len=50, loss=G.LOGISTIC, support=500, **kw):
    return dict({"matrix": "zipf", "n": n, "k": k, "a": a, "mean_len": mean_len, "loss": loss,
                 "support": support}, **kw)


def _bern_case(n, k, density, loss=G.LOGISTIC, support=50, **kw):
    return dict({"matrix": "bernoulli", "n": n, "k": k, "density": density, "loss": loss,
                 "support": support}, **kw)


def _solve(rule, select=1, block=1, lam_ratio=0.1, tol=1e-6, max_epochs=1000, check_every=1, **kw):
    return dict({"kind": "solve", "rule": rule, "select": select, "block": block,
                 "lam_ratio": lam_ratio, "tol": tol, "max_epochs": max_epochs,
                 "check_every": check_every}, **kw)


def listed():
    return [
        # the smallest use: classic cyclic descent on a few thousand entries
        # (one column per iteration, a matrix that fits a cache)
        dict(_bern_case(400, 1000, 0.01), **_solve("cyclic", max_epochs=60), name="cyclic_small"),
        # a small Shotgun problem solved again and again, as in a serving
        # loop or cross-validation: many short iterations
        dict(_bern_case(400, 1000, 0.01), **_solve("shotgun", select=64), name="shotgun_small"),
        # an ordinary Lasso of the small workload's full size
        dict(_bern_case(2000, 5000, 0.01, loss=G.SQUARED),
             **_solve("shotgun", select=96, check_every=0), name="shotgun_lasso_2k"),
        # the repository's main workload: text-like logistic regression
        dict(_zipf_case(100_000, 500_000), **_solve("shotgun", select=4096, lam_ratio=0.05,
                                                    seed=7), name="shotgun_zipf"),
        # the same with the options of the fastest single solve there
        dict(_zipf_case(100_000, 500_000),
             **_solve("shotgun", select=4096, lam_ratio=0.05, seed=7, fused=True, graph=True),
             name="shotgun_zipf_fused_graph"),
        # Thread-Greedy, the paper's best rule, on a mid-size text matrix: two epochs
        dict(_zipf_case(20_000, 100_000, support=100),
             **_solve("thread_greedy", select=1024, block=64, lam_ratio=0.05, tol=0.0,
                      max_epochs=2, seed=7), name="thread_greedy_zipf"),
        # Greedy: every live column proposed for one update, 40 iterations
        dict(_zipf_case(100_000, 500_000),
             **_solve("greedy", lam_ratio=0.05, tol=0.0, max_epochs=40, check_every=0, seed=7),
             name="greedy_zipf"),
        # colouring of the Lasso matrix, and Coloring descent with it
        dict(_zipf_case(200_000, 1_000_000, a=1.2, mean_len=30, loss=G.SQUARED, support=1000),
             kind="color", name="color_zipf"),
        dict(_zipf_case(200_000, 1_000_000, a=1.2, mean_len=30, loss=G.SQUARED, support=1000),
             **_solve("coloring", check_every=0, seed=3), name="coloring_zipf"),
        # a regularisation path on binary data, with the path's fastest options
        dict(_bern_case(50_000, 200_000, 5e-4, support=200, binary=True), kind="path", lambdas=32,
             ratio=0.05, B=16, select=1024, tol=1e-7, max_epochs=2000, improve=10, fused=True,
             epoch=True, name="path_binary"),
        # one large request of the serving stream: |J| from the spectral
        # radius, 25 million entries
        dict(_bern_case(25_000, 100_000, 0.01, loss=G.SQUARED),
             **_solve("shotgun", select=0, lam_ratio=0.2, check_every=0, seed=11, max_epochs=300),
             name="request_25m"),
        # a batch of smaller requests through the server
        {"kind": "server", "n": 8000, "k": 16000, "requests": 6, "mix": 3, "ratio_lo": 0.1,
         "max_epochs": 300, "name": "server_batch"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "small", "zipf", "zipf", "zipf_fused", "thread_greedy", "greedy",
                       "color", "coloring", "path", "request", "server", "check", "check"])
    seed = rng.randrange(1, 1000)
    ratio = round(math.exp(rng.uniform(math.log(0.05), math.log(0.3))), 4)
    if kind == "small":
        n, k = _log(rng, 150, 2000), _log(rng, 300, 5000)
        rule = rng.choice(["cyclic", "shotgun", "shotgun", "stochastic"])
        select = rng.randrange(8, max(9, k // 16)) if rule == "shotgun" else 1
        return dict(_bern_case(n, k, round(rng.uniform(0.005, 0.02), 4),
                               loss=rng.choice([G.LOGISTIC, G.SQUARED])),
                    **_solve(rule, select=select, lam_ratio=max(ratio, 0.1), seed=seed,
                             max_epochs=200 if rule == "shotgun" else max(2, 20_000 // k),
                             check_every=rng.choice([0, 1])))
    n = _log(rng, 5_000, 100_000)
    k = min(500_000, int(n * rng.uniform(2.0, 6.0)) + 1)
    select = rng.choice([512, 1000, 2048, 4096])
    zipf = _zipf_case(n, k, support=rng.randrange(50, 500), mean_len=rng.randrange(20, 50))
    if kind == "zipf":
        return dict(zipf, **_solve("shotgun", select=min(select, k // 64), lam_ratio=ratio,
                                   seed=seed, max_epochs=20, graph=rng.random() < 0.3))
    if kind == "zipf_fused":
        return dict(zipf, **_solve("shotgun", select=min(select, k // 64), lam_ratio=ratio,
                                   seed=seed, max_epochs=30, fused=True, graph=True))
    if kind == "thread_greedy":
        n, k = max(300, n // 5), max(1000, k // 5)
        return dict(dict(zipf, n=n, k=k, support=50),
                    **_solve("thread_greedy", select=rng.choice([512, 1000, 1024]),
                             block=rng.choice([32, 64, 100]), lam_ratio=ratio, tol=0.0,
                             max_epochs=rng.choice([1, 2]), seed=seed))
    if kind == "greedy":
        return dict(zipf, **_solve("greedy", lam_ratio=ratio, tol=0.0,
                                   max_epochs=rng.randrange(10, 40), check_every=0, seed=seed))
    if kind in ("color", "coloring"):
        lasso = _zipf_case(n, k, a=1.2, mean_len=rng.randrange(10, 30), loss=G.SQUARED,
                           support=rng.randrange(50, 1000))
        if kind == "color":
            return dict(lasso, kind="color")
        return dict(lasso, **_solve("coloring", lam_ratio=max(ratio, 0.1), check_every=0,
                                    seed=seed, max_epochs=30))
    if kind == "path":
        n, k = _log(rng, 2_000, 50_000), _log(rng, 8_000, 200_000)
        fused = rng.random() < 0.5
        return dict(_bern_case(n, k, round(25.0 / n, 6), support=100, binary=rng.random() < 0.5,
                               loss=rng.choice([G.LOGISTIC, G.SQUARED])),
                    kind="path", lambdas=rng.randrange(8, 32), ratio=0.1, B=rng.choice([16, 32]),
                    select=rng.choice([128, 256]), tol=1e-7, max_epochs=200,
                    improve=rng.choice([0, 10]), fused=fused, epoch=fused)
    if kind == "request":
        n, k = rng.randrange(1000, 25_000), rng.randrange(1000, 100_000)
        return dict(_bern_case(n, k, round(rng.uniform(0.001, 0.01), 5),
                               loss=rng.choice([G.LOGISTIC, G.SQUARED])),
                    **_solve("shotgun", select=0, lam_ratio=max(ratio, 0.2), check_every=0,
                             seed=seed, max_epochs=100))
    if kind == "server":
        return {"kind": "server", "n": rng.randrange(2000, 8000), "k": rng.randrange(2000, 16000),
                "requests": rng.randrange(2, 6), "mix": seed, "ratio_lo": 0.2, "max_epochs": 200}
    return dict(zipf, kind="check", lam_ratio=ratio, nnz_w=rng.randrange(1, 5000))


# ---------------------------------------------------------------------------
# Preparation and the timed call
# ---------------------------------------------------------------------------
def _matrix(pr):
    return G.Matrix(pr["n"], pr["k"], pr["col_ptr"], pr["row_idx"], pr["val"])


def _params(case, pr, colors=None, num_colors=0):
    flags = (G.FUSED if case.get("fused") else 0) | (G.USE_GRAPH if case.get("graph") else 0)
    if case.get("epoch"):
        flags |= G.FUSED_EPOCH
    return G.make_params(case["loss"], pr["lam"], rule=case.get("rule", "shotgun"),
                         select_size=case["select"], block=case.get("block", 1),
                         seed=case.get("seed", 1), tol=case["tol"],
                         max_epochs=case["max_epochs"], check_every=case.get("check_every", 0),
                         flags=flags, colors=colors, num_colors=num_colors,
                         improve=case.get("improve", 0))


def _check_w(case, pr, seed):
    g = _gen(seed + 77, _dev())
    w = torch.zeros(case["k"], device=_dev())
    at = torch.randperm(case["k"], generator=g, device=_dev())[:case["nnz_w"]]
    w[at] = torch.randn(at.numel(), generator=g, device=_dev())
    return w


def prepare(case, seed):
    kind = case["kind"]
    if kind == "server":
        reqs, seeds = _requests(case, seed)
        st = {"kind": kind, "jobs": []}
        need = 0
        for c, s in zip(reqs, seeds):
            pr = _problem(c, s)
            X, p = _matrix(pr), _params(c, pr)
            need += G.Server.request_bytes(X, p)
            st["jobs"].append((X, pr["y"], p, torch.empty(c["k"], device=_dev()),
                               torch.empty(c["n"], device=_dev())))
        slots = len(reqs)
        st["server"] = G.Server(G.Server.overhead_bytes(slots) + need + 4096, max_slots=slots)
        torch.cuda.synchronize()  # submitted inputs have to be complete
        return st
    pr = _problem(case, seed)
    X = _matrix(pr)
    st = {"kind": kind, "X": X, "y": pr["y"]}
    if kind == "solve":
        colors, nc = G.color(X) if case["rule"] == "coloring" else (None, 0)
        st["colors"] = colors
        st["params"] = _params(case, pr, colors, nc)
        st["ws"] = G.workspace(X, st["params"])
    elif kind == "path":
        t = torch.arange(case["lambdas"], dtype=torch.float64) / (case["lambdas"] - 1)
        st["lambdas"] = (pr["lmax"] * case["ratio"] ** t).numpy()
        st["params"] = _params(case, pr)
        st["B"] = case["B"]
    elif kind == "check":
        st["w"] = _check_w(case, pr, seed)
        st["lam"], st["loss"] = pr["lam"], case["loss"]
        st["ws"] = G.workspace(X)
    return st


def run(st):
    kind = st["kind"]
    if kind == "solve":
        r = G.solve(st["X"], st["y"], st["params"], ws=st["ws"])
        return {"w": r.w, "z": r.z}
    if kind == "color":
        colors, count = G.color(st["X"])
        return {"colors": colors, "count": count}
    if kind == "path":
        r = G.solve_path(st["X"], st["y"], st["params"], st["lambdas"], B=st["B"], want_z=True)
        return {"W": r.W, "Z": r.Z}
    if kind == "check":
        r = G.check(st["X"], st["y"], st["loss"], st["lam"], st["w"], ws=st["ws"])
        return {"objective": r.objective, "kkt": r.kkt, "nnz_w": r.nnz_w, "z64": r.z64,
                "g64": r.g64}
    srv = st["server"]
    for X, y, p, w, z in st["jobs"]:
        srv.submit(X, y, p, w, z)
    left = len(st["jobs"])
    while left:
        left -= len(srv.poll(wait_for=left))
    return {"w": [j[3] for j in st["jobs"]], "z": [j[4] for j in st["jobs"]]}


# ---------------------------------------------------------------------------
# Work
# ---------------------------------------------------------------------------
def _nnz(case):
    if case["matrix"] == "zipf":
        return case["n"] * case["mean_len"]
    return int(case["n"] * case["k"] * case["density"])


def work(case):
    """Inputs read once and outputs written once; the arithmetic of one
    epoch over the matrix (a product, a loss derivative and an update per
    entry: about 16 operations), since how many epochs a solve takes is its
    own result."""
    if case["kind"] == "server":
        parts = [work(dict(c, kind="solve")) for c in _requests(case, 0)[0]]
        return {"bytes": sum(p["bytes"] for p in parts), "flops": sum(p["flops"] for p in parts)}
    nnz, n, k = _nnz(case), case["n"], case["k"]
    bytes_, flops = 8 * nnz + 8 * (k + 1) + 4 * n, 16 * nnz
    if case["kind"] == "color":
        return {"bytes": 4 * nnz + 8 * (k + 1) + 4 * k, "flops": 0}
    if case["kind"] == "path":
        L = case["lambdas"]
        return {"bytes": bytes_ + 4 * L * (n + k), "flops": flops * L}
    if case["kind"] == "check":
        return {"bytes": bytes_ + 4 * k + 8 * (n + k), "flops": 4 * nnz}
    if case["rule"] == "coloring":
        bytes_ += 4 * k
    return {"bytes": bytes_ + 4 * (n + k), "flops": flops}


# ---------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------
def _fin(x):
    x ^= x >> 30
    x = x * 0xBF58476D1CE4E5B9 & _M64
    x ^= x >> 27
    x = x * 0x94D049BB133111EB & _M64
    return x ^ (x >> 31)


def _signed(x):
    return x - (1 << 64) if x >> 63 else x


def _fin_t(x):
    def shr(v, s):
        return (v >> s) & ((1 << (64 - s)) - 1)
    x = x ^ shr(x, 30)
    x = x * _signed(0xBF58476D1CE4E5B9)
    x = x ^ shr(x, 27)
    x = x * _signed(0x94D049BB133111EB)
    return x ^ shr(x, 31)


def _perm(m, seed, epoch, dev):
    """The documented selection permutation: a 4-round Feistel network on the
    next even power of two, cycle-walked into [0, m)."""
    bits = 2
    while (1 << bits) < m:
        bits += 2
    half, mask = bits // 2, (1 << (bits // 2)) - 1
    keys = [_signed(_fin((seed + _GOLD * (epoch * 8 + r + 1)) & _M64)) for r in range(4)]
    x = torch.arange(m, device=dev)
    todo = torch.arange(m, device=dev)
    while todo.numel():
        v = x[todo]
        a, b = v >> half, v & mask
        for key in keys:
            a, b = b, a ^ (_fin_t(b ^ key) & mask)
        v = (a << half) | b
        x[todo] = v
        todo = todo[v >= m]
    return x


class _Ref:
    """Algorithm 1 in FP64 with plain torch."""

    def __init__(self, pr, loss, dev):
        self.n, self.k, self.loss, self.lam = pr["n"], pr["k"], loss, pr["lam"]
        self.ptr = pr["col_ptr"].to(dev)
        self.rows = pr["row_idx"].to(dev).long()
        self.val = pr["val"].to(dev).double()
        self.y = pr["y"].to(dev).double()
        self.lens = self.ptr[1:] - self.ptr[:-1]
        self.dev = dev
        self.cid = torch.repeat_interleave(torch.arange(self.k, device=dev), self.lens)
        self.ss = _segsum(self.val * self.val, self.ptr)
        self.c = self.ss * ((1.0 if loss == G.SQUARED else 0.25) / self.n)
        self.live = torch.nonzero(self.lens).reshape(-1)

    def zeros(self, m):
        return torch.zeros(m, dtype=torch.float64, device=self.dev)

    def dloss(self, y, t):
        return t - y if self.loss == G.SQUARED else -y * torch.sigmoid(-y * t)

    def product(self, w):
        return self.zeros(self.n).index_add_(0, self.rows, self.val * w[self.cid])

    def tproduct(self, r):
        return _segsum(self.val * r[self.rows], self.ptr)

    def check(self, w):
        z = self.product(w)
        g = self.tproduct(self.dloss(self.y, z)) / self.n
        v = torch.where(w != 0, (g + self.lam * torch.sign(w)).abs(),
                        (g.abs() - self.lam).clamp(min=0))
        m = self.y * z
        f = 0.5 * (self.y - z) ** 2 if self.loss == G.SQUARED else \
            torch.nn.functional.softplus(-m, threshold=1e9)
        obj = float(f.sum()) / self.n + self.lam * float(w.abs().sum())
        return z, g, float(v.max()), obj

    def pstar(self):
        d = torch.where(self.ss > 0, self.ss.clamp(min=1e-300).rsqrt(), self.zeros(self.k))
        v = torch.where(self.ss > 0, 1.0, 0.0).double()
        v /= v.norm()
        for _ in range(20):
            v = d * self.tproduct(self.product(d * v))
            rho = float(v.norm())
            v /= rho
        kl = self.live.numel()
        return max(1, min(kl, int(kl / (2 * rho)))) if rho > 0 else 1

    def solve(self, case):
        rule, n = case["rule"], self.n
        kl = self.live.numel()
        S = {"cyclic": 1, "stochastic": 1, "greedy": kl}.get(rule, case["select"])
        S = max(1, min(S if S > 0 else self.pstar(), kl))
        w, z = self.zeros(self.k), self.zeros(n)
        nxt, epoch = 1, 0
        while epoch < case["max_epochs"]:
            order = self.live if rule == "cyclic" else \
                self.live[_perm(kl, case.get("seed", 1), epoch, self.dev)]
            ln = self.lens[order]
            off = torch.zeros(kl + 1, dtype=torch.int64, device=self.dev)
            torch.cumsum(ln, 0, out=off[1:])
            pos = torch.repeat_interleave(torch.arange(kl, device=self.dev), ln)
            ent = torch.arange(pos.numel(), device=self.dev) - off[pos] + self.ptr[order][pos]
            rr, vv, cc = self.rows[ent], self.val[ent], self.c[order]
            cut = off[torch.arange(0, kl + S, S, device=self.dev).clamp(max=kl)].tolist()
            for t in range((kl + S - 1) // S):
                p0, p1 = t * S, min(kl, t * S + S)
                r, v, seg = rr[cut[t]:cut[t + 1]], vv[cut[t]:cut[t + 1]], pos[cut[t]:cut[t + 1]] - p0
                j, c = order[p0:p1], cc[p0:p1]
                g = _segsum(v * self.dloss(self.y[r], z[r]), off[p0:p1 + 1] - cut[t]) / n
                wj = w[j]
                d = -torch.minimum(torch.maximum(wj, (g - self.lam) / c), (g + self.lam) / c)
                if rule in ("greedy", "thread_greedy"):
                    phi = 0.5 * c * d * d + g * d + self.lam * ((wj + d).abs() - wj.abs())
                    B = p1 - p0 if rule == "greedy" else case["block"]
                    pad = -(p1 - p0) % B
                    blk = torch.nn.functional.pad(phi, (0, pad), value=math.inf).reshape(-1, B)
                    low = blk.min(1, keepdim=True)[0]
                    first = torch.where(blk == low, torch.arange(B, device=self.dev), B).min(1)[0]
                    keep = torch.zeros_like(blk)
                    keep[torch.arange(blk.shape[0], device=self.dev), first] = 1.0
                    d = d * keep.reshape(-1)[:p1 - p0]
                w[j] = wj + d
                z.index_add_(0, r, v * d[seg])
            epoch += 1
            if epoch >= nxt or epoch == case["max_epochs"]:
                ce = case["check_every"]
                nxt = epoch + (ce if ce > 0 else min(64, max(1, epoch // 10)))
                z, _, kkt, _ = self.check(w)
                if kkt <= case["tol"]:
                    break
        return {"w": w, "z": self.product(w)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "server":
        out = [_exact_solve(c, s) for c, s in zip(*_requests(case, seed))]
        return {"w": [o["w"] for o in out], "z": [o["z"] for o in out]}
    if kind == "check":
        pr = _problem(case, seed)
        w = _check_w(case, pr, seed).double()
        z, g, kkt, obj = _Ref(pr, case["loss"], _dev()).check(w)
        return {"objective": obj, "kkt": kkt, "nnz_w": int((w != 0).sum()), "z64": z, "g64": g}
    # asynchronous updates have no defined trajectory, a colouring in plain
    # Python takes minutes, and the colours of a Coloring solve come from it
    if kind != "solve" or case.get("fused") or case["rule"] == "coloring":
        return None
    return _exact_solve(case, seed)


def _exact_solve(case, seed):
    pr = _problem(case, seed)
    # one column per window: thousands of tiny steps, cheaper on the host
    tiny = case["rule"] in ("cyclic", "stochastic")
    return _Ref(pr, case["loss"], "cpu" if tiny else _dev()).solve(case)
