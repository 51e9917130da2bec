"""The calls that a program built on this library spends its time in, as cases
that can be timed and checked.

Eight families, each through the public entry points of ``ops`` and ``batch``
and each with its return sweep: the linear-recurrence scan, reduce_by_index,
the planned scatter, the Gaussian-mixture log-likelihood, the segmented batch
of scan and sum VJPs, the scan and reduce_by_index with a general operator,
and a Newton step of k-means.  ``exact`` gives the same outputs in 64 bits
from plain torch (recurrences by recursive doubling, sums by index_add).
"""
from __future__ import annotations

import math

import torch

from paper_2202_10297_amd import ops
from paper_2202_10297_amd.batch import SegPlan

_DTYPES = {"f32": torch.float32, "f64": torch.float64}
_SIZE = {"f32": 4, "f64": 8}
_NCOMP = {"logaddexp": 1, "linrec": 2, "mat2": 4}


def listed():
    return [
        # the scan's own configuration: 65,536 FP64 pairs, where launches and latency count
        {"name": "scan_65536_f64", "kind": "scan", "n": 65536, "dtype": "f64"},
        # the long end of the scan's sweep, bound by memory
        {"name": "scan_2e26_f64", "kind": "scan", "n": 1 << 26, "dtype": "f64"},
        # the histogram configuration: bins beyond one LDS, uniform indices, sums
        {"name": "hist_add_2e26_m2e16", "kind": "hist", "op": "add", "n": 1 << 26, "m": 1 << 16, "dist": "uniform",
         "dtype": "f32"},
        # the same with extremes, a million bins and the skew of word counts
        {"name": "hist_max_2e26_m2e20_zipf", "kind": "hist", "op": "max", "n": 1 << 26, "m": 1 << 20, "dist": "zipf",
         "dtype": "f32"},
        # a request of the serving mix: a ragged million elements, a few thousand bins
        {"name": "hist_add_1000003_m4099", "kind": "hist", "op": "add", "n": 1000003, "m": 4099, "dist": "zipf",
         "dtype": "f32"},
        # the scatter configuration: 2^24 unique targets in 2^26 elements
        {"name": "scatter_2e24_into_2e26", "kind": "scatter", "n": 1 << 26, "m": 1 << 24, "dtype": "f32"},
        # the mixture configuration: one gradient step over a million points
        {"name": "gmm_1e6_d64_k200", "kind": "gmm", "N": 1000000, "D": 64, "K": 200},
        # a mixture request of the serving mix
        {"name": "gmm_10007_d32_k50", "kind": "gmm", "N": 10007, "D": 32, "K": 50},
        # 4,096 scans and sums of uneven lengths in one launch each way
        {"name": "batch_4096_f32", "kind": "batch", "segments": 4096, "lo": 64, "hi": 1 << 20, "lengths_seed": 0},
        # a scan of 2x2 matrix products (chains of linear maps), a ragged length
        {"name": "scan_mat2_20000003_f32", "kind": "scan_generic", "op": "mat2", "n": 20000003, "dtype": "f32"},
        # per-bin recurrences in index order: an operator that does not commute
        {"name": "hist_linrec_2e24_m2e16", "kind": "hist_generic", "op": "linrec", "n": 1 << 24, "m": 1 << 16,
         "dist": "uniform", "dtype": "f32"},
        # one Newton step of k-means with many centres
        {"name": "kmeans_10000_d256_k1024", "kind": "kmeans", "N": 10000, "D": 256, "K": 1024},
    ]


def _logu(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))) | (1 if rng.random() < 0.7 else 0)


def draw(rng):
    kind = rng.choice(["scan", "scan", "hist", "hist", "hist", "scatter", "gmm", "gmm", "batch", "scan_generic",
                       "hist_generic", "kmeans"])
    if kind == "scan":
        dt = rng.choice(["f64", "f32"])
        return {"kind": kind, "n": min(_logu(rng, 1000, 1 << 26), 1 << 26), "dtype": dt}
    if kind == "hist":
        op, dt = rng.choice(["add", "add", "max", "min", "mul"]), rng.choice(["f32", "f32", "f64"])
        m = min(_logu(rng, 1 << 10, 1 << 20), 1 << 20)
        dist = "uniform" if op == "mul" else rng.choice(["uniform", "zipf"])
        n = _logu(rng, 10000, min(1 << 25, 2048 * m) if op == "mul" else 1 << 26 if dt == "f32" else 1 << 25)
        return {"kind": kind, "op": op, "n": min(n, 1 << 26), "m": m, "dist": dist, "dtype": dt}
    if kind == "scatter":
        m = min(_logu(rng, 100000, 1 << 24), 1 << 24)
        return {"kind": kind, "n": min(int(m * rng.uniform(1.5, 8.0)), 1 << 26), "m": m,
                "dtype": rng.choice(["f32", "f32", "f64"])}
    if kind == "gmm":
        D, K = rng.choice([(32, 50), (32, 200), (64, 25), (64, 200), (64, 101)])
        return {"kind": kind, "N": min(_logu(rng, 1000, 1000000), 1000000), "D": D, "K": K}
    if kind == "batch":
        return {"kind": kind, "segments": _logu(rng, 64, 4096) & ~1, "lo": 64, "hi": 1 << 20,
                "lengths_seed": rng.randrange(1000)}
    if kind == "scan_generic":
        return {"kind": kind, "op": rng.choice(["logaddexp", "linrec", "mat2"]), "n": _logu(rng, 10000, 20000000),
                "dtype": rng.choice(["f32", "f64"])}
    if kind == "hist_generic":
        return {"kind": kind, "op": rng.choice(["linrec", "mat2"]), "n": min(_logu(rng, 100000, 1 << 24), 1 << 24),
                "m": min(_logu(rng, 1 << 8, 1 << 18), 1 << 18), "dist": rng.choice(["uniform", "zipf"]),
                "dtype": "f32"}
    K, D = _logu(rng, 5, 1024), rng.choice([2, 16, 35, 64, 128, 256])
    return {"kind": kind, "N": max(K, min(_logu(rng, 2000, 494019), (10000 * 256 * 1024) // (K * D))), "D": D, "K": K}


# ------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape, dtype=torch.float32):
    return torch.randn(*shape, dtype=dtype, device="cuda", generator=g)


def _indices(g, n, m, dist):
    """Bin indices in [0, m): uniform, or Zipf(1.1) ranks through a permutation."""
    if dist == "uniform":
        return torch.randint(0, m, (n,), dtype=torch.int32, device="cuda", generator=g)
    cdf = torch.cumsum(torch.arange(1, m + 1, dtype=torch.float64, device="cuda") ** -1.1, 0)
    u = torch.rand(n, dtype=torch.float64, device="cuda", generator=g) * cdf[-1]
    rank = torch.searchsorted(cdf, u, right=True).clamp_(max=m - 1)
    return torch.randperm(m, device="cuda", generator=g)[rank].to(torch.int32)


def _components(g, op, n, dt):
    """Elements of a general operator; 2x2 factors are rotations, half of them
    reflected, so that long products stay orthogonal."""
    if op == "logaddexp":
        return [_randn(g, n, dtype=dt)]
    if op == "linrec":
        return [torch.rand(n, dtype=dt, device="cuda", generator=g) * 0.5 + 0.5, _randn(g, n, dtype=dt)]
    th = (torch.rand(n, dtype=torch.float64, device="cuda", generator=g) * 2 - 1) * math.pi
    f = (torch.rand(n, device="cuda", generator=g) < 0.5).double() * 2 - 1
    c, s = th.cos(), th.sin()
    return [t.to(dt) for t in (c, -s * f, s, c * f)]


def _lengths(case):
    g = torch.Generator()
    g.manual_seed(case["lengths_seed"])
    u = torch.rand(case["segments"], dtype=torch.float64, generator=g)
    lo, hi = math.log(case["lo"]), math.log(case["hi"])
    return torch.exp(lo + u * (hi - lo)).floor().to(torch.int64)


def _inputs(case, seed):
    g, kind = _gen(seed), case["kind"]
    if kind == "scan":
        n, dt = case["n"], _DTYPES[case["dtype"]]
        return {"a": torch.rand(n, dtype=dt, device="cuda", generator=g) * 0.5 + 0.5, "b": _randn(g, n, dtype=dt),
                "yA": _randn(g, n, dtype=dt), "yB": _randn(g, n, dtype=dt)}
    if kind == "hist":
        n, m, dt = case["n"], case["m"], _DTYPES[case["dtype"]]
        vs = _randn(g, n, dtype=dt)
        if case["op"] == "mul":  # factors near +-1 and a few zeros, so that products stay in range
            zero = torch.rand(n, device="cuda", generator=g) < 0.25 * m / n
            vs = torch.where(zero, torch.zeros_like(vs), torch.exp(0.02 * vs) * torch.sign(_randn(g, n, dtype=dt)))
        return {"inds": _indices(g, n, m, case["dist"]), "vs": vs, "hs_bar": _randn(g, m, dtype=dt)}
    if kind == "scatter":
        n, m, dt = case["n"], case["m"], _DTYPES[case["dtype"]]
        return {"xs": _randn(g, n, dtype=dt), "is_": torch.randperm(n, device="cuda", generator=g)[:m].to(torch.int32),
                "vs": _randn(g, m, dtype=dt), "ys_bar": _randn(g, n, dtype=dt)}
    if kind == "gmm":
        N, D, K = case["N"], case["D"], case["K"]
        return {"X": _randn(g, N, D), "alpha": _randn(g, K), "mu": _randn(g, K, D), "q": 0.1 * _randn(g, K, D),
                "l": 0.1 * _randn(g, K, D * (D - 1) // 2)}
    if kind == "batch":
        total = int(_lengths(case).sum())
        return {"a": torch.rand(total, device="cuda", generator=g) * 0.5 + 0.5, "b": _randn(g, total),
                "yA": _randn(g, total), "yB": _randn(g, total), "sum_ybar": _randn(g, case["segments"])}
    if kind == "scan_generic":
        n, dt = case["n"], _DTYPES[case["dtype"]]
        xs = _components(g, case["op"], n, dt)
        return {"xs": xs, "y_bar": [_randn(g, n, dtype=dt) for _ in xs]}
    if kind == "hist_generic":
        n, m, dt = case["n"], case["m"], _DTYPES[case["dtype"]]
        xs = _components(g, case["op"], n, dt)
        return {"inds": _indices(g, n, m, case["dist"]), "xs": xs, "hs_bar": [_randn(g, m, dtype=dt) for _ in xs]}
    N, D, K = case["N"], case["D"], case["K"]
    lab = torch.randint(0, K, (N,), device="cuda", generator=g)
    X = (3.0 * _randn(g, K, D))[lab] + _randn(g, N, D)
    return {"X": X, "C": X[torch.randperm(N, device="cuda", generator=g)[:K]].clone()}


def prepare(case, seed):
    st = {"case": case, **_inputs(case, seed)}
    if case["kind"] == "batch":
        st["plan"] = SegPlan(_lengths(case).numpy(), dtype=torch.float32)
    if case["kind"] == "scatter":
        # the target array and its adjoint are overwritten: what the upstream sweep hands over is kept apart
        st["upstream"], st["ys_bar"] = st["ys_bar"], torch.empty_like(st["ys_bar"])
    if case["kind"] == "kmeans":
        st["ones"] = torch.ones_like(st["C"])
    return st


# --------------------------------------------------------------------- pass
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "scan":
        A, B, ck = ops.linrec_scan(st["a"], st["b"])
        a_bar, b_bar = ops.linrec_scan_vjp(st["a"], st["b"], st["yA"], st["yB"], ckpt=ck)
        return {"A": A, "B": B, "a_bar": a_bar, "b_bar": b_bar}
    if kind == "hist":
        hs, aux = ops.hist(case["op"], st["inds"], st["vs"], case["m"])
        return {"hs": hs, **aux, "vs_bar": ops.hist_vjp(case["op"], st["inds"], st["vs"], case["m"], aux,
                                                        st["hs_bar"])}
    if kind == "scatter":
        plan = ops.scatter_planned_(st["xs"], st["is_"], st["vs"])
        st["ys_bar"].copy_(st["upstream"])
        vs_bar = ops.scatter_planned_vjp_(st["ys_bar"], case["m"], plan)
        return {"ys": st["xs"], "vs_bar": vs_bar, "xs_bar": st["ys_bar"]}
    if kind == "gmm":
        P = (st["X"], st["alpha"], st["mu"], st["q"], st["l"])
        ll, lse = ops.gmm_objective(*P)
        grads = ops.gmm_vjp(*P, lse=lse)
        return {"loglik": ll, "alpha_bar": grads[0], "mu_bar": grads[1], "q_bar": grads[2], "l_bar": grads[3]}
    if kind == "batch":
        A, B, ck = st["plan"].scan(st["a"], st["b"])
        a_bar, b_bar, x_bar = st["plan"].vjp(st["a"], st["b"], st["yA"], st["yB"], ckpt=ck, sum_ybar=st["sum_ybar"])
        return {"A": A, "B": B, "a_bar": a_bar, "b_bar": b_bar, "sum_xbar": x_bar}
    if kind == "scan_generic":
        ys, ck = ops.scan_generic(case["op"], st["xs"])
        return {"ys": ys, "x_bar": ops.scan_generic_vjp(case["op"], st["xs"], st["y_bar"], ckpt=ck)}
    if kind == "hist_generic":
        hs = ops.hist_generic(case["op"], st["inds"], st["xs"], case["m"])
        return {"hs": hs, "x_bar": ops.hist_generic_vjp(case["op"], st["inds"], st["xs"], st["hs_bar"])}
    f, assign = ops.kmeans_objective(st["X"], st["C"])
    c_bar, diag = ops.kmeans_vjp(st["X"], st["C"], assign, C_dot=st["ones"])
    return {"f": f, "assign": assign, "c_bar": c_bar, "diag": diag}


def work(case):
    kind = case["kind"]
    s = _SIZE.get(case.get("dtype", "f32"))
    if kind == "scan":  # a, b in, A, B out; a, b and the adjoints in, two adjoints out
        return {"bytes": 10 * s * case["n"], "flops": 11 * case["n"]}
    if kind == "hist":
        n, m = case["n"], case["m"]
        back = {"add": 4 + s, "mul": 4 + 2 * s}.get(case["op"], s)
        return {"bytes": n * (4 + s + back) + m * (2 * s + 8), "flops": 2 * n}
    if kind == "scatter":  # index, value, overwritten value; index, adjoint, zero, adjoint; the upstream adjoint once
        return {"bytes": case["m"] * (2 * 4 + 6 * s) + 2 * s * case["n"], "flops": 0}
    if kind == "gmm":  # the triangular products of the objective and the contraction of its adjoint
        N, D, K = case["N"], case["D"], case["K"]
        return {"bytes": 2 * 4 * N * D + 16 * N + 3 * 4 * K * (D * (D + 3) // 2), "flops": 2 * N * K * D * (D + 1)}
    if kind == "batch":
        total = int(_lengths(case).sum())
        return {"bytes": 44 * total, "flops": 11 * total}
    if kind == "scan_generic":
        k = _NCOMP[case["op"]]
        return {"bytes": 5 * k * s * case["n"], "flops": {1: 12, 2: 11, 4: 48}[k] * case["n"]}
    if kind == "hist_generic":
        n, m, k = case["n"], case["m"], _NCOMP[case["op"]]
        return {"bytes": n * (8 + 3 * k * s) + 2 * m * k * s, "flops": {2: 12, 4: 60}[k] * n}
    N, D, K = case["N"], case["D"], case["K"]
    return {"bytes": 2 * 4 * N * D + 8 * N + 5 * 4 * K * D, "flops": 2 * N * K * D}


# ------------------------------------------------------------ 64-bit answers
def _mul2(x, y):
    return [x[0] * y[0] + x[1] * y[2], x[0] * y[1] + x[1] * y[3],
            x[2] * y[0] + x[3] * y[2], x[2] * y[1] + x[3] * y[3]]


def _linrec(x, y):
    return [y[0] * x[0], y[0] * x[1] + y[1]]


def _rows(x, y):
    """Two row vectors u under an affine map v -> v M + u, packed (u, u', M); x is applied first."""
    return [x[0] * y[4] + x[1] * y[6] + y[0], x[0] * y[5] + x[1] * y[7] + y[1],
            x[2] * y[4] + x[3] * y[6] + y[2], x[2] * y[5] + x[3] * y[7] + y[3], *_mul2(x[4:], y[4:])]


def _scan(comb, xs, head=None):
    """Inclusive scan by doubling; head[i] is the first index of i's segment."""
    n, d = xs[0].numel(), 1
    at = torch.arange(n, device=xs[0].device) if head is not None else None
    most = n if head is None else int((at - head).max()) + 1 if n else 0
    while d < most:
        got = comb([x[:-d] for x in xs], [x[d:] for x in xs])
        if head is not None:
            inside = at[d:] - d >= head[d:]
            got = [torch.where(inside, y, x[d:]) for x, y in zip(xs, got)]
        xs = [torch.cat([x[:d], y]) for x, y in zip(xs, got)]
        d *= 2
    return xs


def _back(comb, xs, last=None):
    """The scan from the right, later elements first; last[i] is the last index of i's segment."""
    n = xs[0].numel()
    head = None if last is None else n - 1 - last.flip(0)
    return [x.flip(0) for x in _scan(comb, [x.flip(0) for x in xs], head)]


def _before(x, first, fill):
    """x one place to the right, `fill` where a segment begins."""
    return torch.where(first, torch.full_like(x, fill), torch.roll(x, 1))


def _linrec_adjoint(a, yA, yB, A, B, head, last):
    at = torch.arange(a.numel(), device=a.device)
    first, end = at == head, at == last
    nxt = torch.where(end, torch.zeros_like(a), torch.roll(a, -1))
    rA, rB = _back(_linrec, [nxt, yA], last)[1], _back(_linrec, [nxt, yB], last)[1]
    return rA * _before(A, first, 1.0) + rB * _before(B, first, 0.0), rB


def _linrec_exact(a, b, yA, yB, head=None, last=None):
    n = a.numel()
    if head is None:
        head = torch.zeros(n, dtype=torch.int64, device=a.device)
        last = torch.full_like(head, n - 1)
    A, B = _scan(_linrec, [a, b], head)
    return [A, B, *_linrec_adjoint(a, yA, yB, A, B, head, last)]


def _exact_scan_generic(op, xs, yb):
    n = xs[0].numel()
    if op == "linrec":
        A, B, ab, bb = _linrec_exact(*xs, *yb)
        return {"ys": [A, B], "x_bar": [ab, bb]}
    if op == "logaddexp":
        y = torch.logcumsumexp(xs[0], 0)
        r = torch.cumsum((yb[0] * torch.exp(-y)).flip(0), 0).flip(0)
        return {"ys": [y], "x_bar": [r * torch.exp(xs[0])]}
    ys = _scan(_mul2, xs)
    # r_i = y_bar_i + r_{i+1} X_{i+1}^T
    nxt = [torch.cat([x[1:], x.new_zeros(1)]) for x in (xs[0], xs[2], xs[1], xs[3])]
    r = _back(_rows, [*yb, *nxt])[:4]
    p = [torch.cat([y.new_full((1,), e), y[:-1]]) for y, e in zip(ys, (1.0, 0.0, 0.0, 1.0))]
    return {"ys": ys, "x_bar": _mul2([p[0], p[2], p[1], p[3]], r)}


def _exact_hist_generic(op, inds, xs, hb, m):
    n = inds.numel()
    order = torch.sort(inds, stable=True).indices
    key = inds[order].to(torch.int64)
    s = [x[order] for x in xs]
    head, last = torch.searchsorted(key, key), torch.searchsorted(key, key, right=True) - 1
    at = torch.arange(n, device=inds.device)
    comb = {"linrec": _linrec, "mat2": _mul2}[op]
    pre = _scan(comb, s, head)
    suf = _back(lambda x, y: comb(y, x), s, last)
    ident = {"linrec": (1.0, 0.0), "mat2": (1.0, 0.0, 0.0, 1.0)}[op]
    hs = [torch.full((m,), e, dtype=torch.float64, device=inds.device) for e in ident]
    end = at == last
    for h, p in zip(hs, pre):
        h[key[end]] = p[end]
    l = [_before(p, at == head, e) for p, e in zip(pre, ident)]
    r = [torch.where(end, torch.full_like(x, e), torch.roll(x, -1)) for x, e in zip(suf, ident)]
    y = [h[key] for h in hb]
    if op == "linrec":
        xb = [r[0] * (y[0] * l[0] + y[1] * l[1]), r[0] * y[1]]
    else:  # l^T y_bar r^T
        xb = _mul2(_mul2([l[0], l[2], l[1], l[3]], y), [r[0], r[2], r[1], r[3]])
    return {"hs": hs, "x_bar": [torch.empty_like(x).index_put_((order,), x) for x in xb]}


def _exact_gmm(X, alpha, mu, q, l):
    N, D = X.shape
    K = alpha.numel()
    low = torch.tril_indices(D, D, -1, device=X.device)
    s = torch.empty(K, N, dtype=torch.float64, device=X.device)
    Q = torch.diag_embed(torch.exp(q))
    Q[:, low[0], low[1]] = l
    for k in range(K):
        z = (X - mu[k]) @ Q[k].t().contiguous()
        s[k] = alpha[k] + q[k].sum() - 0.5 * (z * z).sum(1)
    lse = torch.logsumexp(s, 0)
    ll = lse.sum() - N * torch.logsumexp(alpha, 0) - 0.5 * N * D * math.log(2 * math.pi)
    w = torch.exp(s - lse)
    W = w.sum(1)
    mb, qb, lb = torch.empty_like(mu), torch.empty_like(q), torch.empty_like(l)
    for k in range(K):
        y = X - mu[k]
        z = y @ Q[k].t().contiguous()
        wz = w[k][:, None] * z
        G = wz.t().contiguous() @ y
        mb[k] = Q[k].t().contiguous() @ wz.sum(0)
        qb[k] = W[k] - torch.exp(q[k]) * torch.diagonal(G)
        lb[k] = -G[low[0], low[1]]
    return {"loglik": ll.reshape(1), "alpha_bar": W - N * torch.softmax(alpha, 0), "mu_bar": mb, "q_bar": qb,
            "l_bar": lb}


def exact(case, seed):
    kind = case["kind"]
    x = {k: [t.double() for t in v] if isinstance(v, list) else v.double() if v.is_floating_point() else v
         for k, v in _inputs(case, seed).items()}
    if kind == "scan":
        return dict(zip(("A", "B", "a_bar", "b_bar"), _linrec_exact(x["a"], x["b"], x["yA"], x["yB"])))
    if kind == "batch":
        L = _lengths(case).to(x["a"].device)
        ends = torch.cumsum(L, 0)
        head, last = torch.repeat_interleave(ends - L, L), torch.repeat_interleave(ends - 1, L)
        A, B, ab, bb = _linrec_exact(x["a"], x["b"], x["yA"], x["yB"], head, last)
        return {"A": A, "B": B, "a_bar": ab, "b_bar": bb, "sum_xbar": torch.repeat_interleave(x["sum_ybar"], L)}
    if kind == "scatter":
        i = x["is_"].to(torch.int64)
        ys, xb = x["xs"].clone(), x["ys_bar"].clone()
        ys[i], xb[i] = x["vs"], 0.0
        return {"ys": ys, "vs_bar": x["ys_bar"][i], "xs_bar": xb}
    if kind == "hist":
        m, i, vs, hb = case["m"], x["inds"].to(torch.int64), x["vs"], x["hs_bar"]
        if case["op"] == "add":
            return {"hs": torch.zeros_like(hb).index_add_(0, i, vs), "vs_bar": hb[i]}
        if case["op"] == "mul":
            z = torch.bincount(i[vs == 0], minlength=m)
            p = torch.ones_like(hb).scatter_reduce_(0, i, torch.where(vs == 0, torch.ones_like(vs), vs), "prod")
            rest = torch.where(vs == 0, (z[i] == 1) * p[i], (z[i] == 0) * p[i] / vs)
            return {"hs": torch.where(z == 0, p, torch.zeros_like(p)), "p": p, "z": None, "vs_bar": hb[i] * rest}
        worst = -math.inf if case["op"] == "max" else math.inf
        hs = torch.full_like(hb, worst).scatter_reduce_(0, i, vs, "amax" if case["op"] == "max" else "amin")
        at = torch.arange(i.numel(), device=i.device)
        won = vs == hs[i]
        who = torch.full((m,), i.numel(), device=i.device).scatter_reduce_(0, i[won], at[won], "amin")
        vb, some = torch.zeros_like(vs), who < i.numel()
        vb[who[some]] = hb[some]
        return {"hs": hs, "winner": None, "vs_bar": vb}
    if kind == "gmm":
        return _exact_gmm(x["X"], x["alpha"], x["mu"], x["q"], x["l"])
    if kind == "scan_generic":
        return _exact_scan_generic(case["op"], x["xs"], x["y_bar"])
    if kind == "hist_generic":
        return _exact_hist_generic(case["op"], x["inds"], x["xs"], x["hs_bar"], case["m"])
    X, C = x["X"], x["C"]
    N, (K, D) = X.shape[0], C.shape
    best = torch.full((N,), math.inf, dtype=torch.float64, device=X.device)
    who = torch.zeros(N, dtype=torch.int64, device=X.device)
    for k in range(K):
        d = (X - C[k]).square().sum(1)
        near = d < best
        best, who = torch.where(near, d, best), torch.where(near, torch.full_like(who, k), who)
    cnt = torch.bincount(who, minlength=K).double()[:, None]
    S = torch.zeros_like(C).index_add_(0, who, X)
    return {"f": best.sum().reshape(1), "assign": None, "c_bar": 2 * (cnt * C - S), "diag": 2 * cnt.expand(K, D)}
