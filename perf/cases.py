"""The workloads whose speed counts: calls of the public entry points over the
range of sizes, types and options that they are used with.

A case is a dict of plain values. ``path`` names the entry point:

``pdist``    distance matrix of one collection (``p``; ``p = 0``: L2 Gram matrix)
``window``   rows of a larger matrix (one worker's share of a big collection)
``cdist``    one collection against another (test against training curves)
``batched``  many small independent collections in one launch
``grad``     matrix and its gradient with respect to every time and value
``ranged``   distances over a time range with an exponential time weight
``reduce``   mean, std, max, ... curve of groups of a collection
``combine``  index by index combination of two collections
``norms``    one L_p norm per curve

``n`` is the number of PCFs, ``lo`` and ``hi`` bound the rows of each
(uniformly drawn), ``dtype`` is "f32" or "f64", ``shape`` the kind of curve:
"walk" (gaps Exp(1), values N(0,1)), "rank" (nonincreasing integers, like
stable ranks of persistence modules, with many breakpoints that do not change
the value) or "grid" (curves sampled at common times).
"""
import math

import numpy as np
import torch

from paper_2404_07183_amd import api

_DT = {"f32": np.float32, "f64": np.float64}
_ESZ = {"f32": 4, "f64": 8}


def _case(path, n, lo, hi, dtype="f64", name=None, **kw):
    c = {"path": path, "n": n, "lo": lo, "hi": hi, "dtype": dtype, "shape": "walk", "p": 1.0}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # A notebook user's first matrix (the small plain configuration): the
        # whole call, planning and launches included, is latency.
        _case("pdist", 200, 10, 100, name="l1_f64_n200"),
        # A kernel matrix for a classifier on about a thousand curves: not a
        # multiple of anything, one or two waves of workgroups.
        _case("pdist", 1001, 20, 300, p=0.0, name="gram_f64_n1001"),
        # L2 distances in single precision at medium size.
        _case("pdist", 3000, 50, 500, dtype="f32", p=2.0, name="l2_f32_n3000"),
        # General p (the user guide's 3.5): arithmetic beside the merge.
        _case("pdist", 1500, 50, 300, p=3.5, name="l35_f64_n1500"),
        # The plain configuration, the headline workload: the largest call.
        _case("pdist", 20000, 50, 500, name="l1_f64_n20000"),
        # A chunk of one worker's strip of a big stable-rank matrix: long
        # curves in single precision, a window away from the diagonal.
        _case("window", 12000, 100, 1000, dtype="f32", shape="rank", rows=1500,
              name="l1_f32_strip_1500x12000"),
        # Test curves against training curves, both counts odd.
        _case("cdist", 301, 50, 500, m=5003, name="cdist_l1_f64_301x5003"),
        # Many independent collections (bootstrap folds, classes): sizes over
        # two decades, row counts geometric with one-row and very long curves.
        _case("batched", 128, 1, 5000, p=2.0, smin=16, smax=1024, mean=200,
              name="batched_l2_f64_b128"),
        # One training step's matrix and gradient, forward and backward.
        _case("grad", 2048, 20, 300, p=2.0, power=True, name="grad_l2sq_f64_n2048"),
        # Early times weighted more, over a range (restriction, time warp, matrix).
        _case("ranged", 5000, 50, 500, a=2.5, b=40.0, c=0.1, name="ranged_l1_f64_n5000"),
        # The mean curve of a whole collection, then per-class standard
        # deviations: a deep tree, and many shallow ones.
        _case("reduce", 20000, 50, 500, op="mean", group=20000, name="mean_f64_n20000"),
        _case("reduce", 20000, 50, 500, op="std", group=20, name="std_f64_1000x20"),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["pdist", "pdist", "pdist", "window", "cdist", "batched", "grad",
                       "ranged", "reduce", "reduce", "combine", "norms"])
    dtype = rng.choice(["f32", "f64"])
    shape = rng.choice(["walk", "walk", "rank"])
    lo = _logint(rng, 2, 200)
    hi = lo + _logint(rng, 8, 800)
    if path == "pdist":
        return _case(path, _logint(rng, 50, 6000), lo, hi, dtype, shape=shape,
                     p=rng.choice([0.0, 1.0, 1.0, 2.0, 2.0, 3.0, 1.5]))
    if path == "window":
        n = _logint(rng, 500, 12000)
        return _case(path, n, lo, hi, dtype, shape=shape, rows=_logint(rng, 16, n // 4),
                     p=rng.choice([1.0, 2.0]))
    if path == "cdist":
        return _case(path, _logint(rng, 4, 1000), lo, hi, dtype, shape=shape,
                     m=_logint(rng, 50, 6000), p=rng.choice([0.0, 1.0, 2.0]))
    if path == "batched":
        return _case(path, _logint(rng, 8, 256), 1, 5000, dtype, p=rng.choice([0.0, 1.0, 2.0]),
                     smin=_logint(rng, 4, 32), smax=_logint(rng, 64, 700),
                     mean=_logint(rng, 20, 200))
    if path == "grad":
        return _case(path, _logint(rng, 50, 2500), lo, min(hi, 500), dtype,
                     power=rng.choice([False, True]), p=rng.choice([0.0, 1.0, 2.0])) \
            if lo < 400 else _case(path, 333, 20, 300, dtype, power=True, p=2.0)
    if path == "ranged":
        return _case(path, _logint(rng, 100, 5000), lo, hi, dtype, a=rng.uniform(0.5, 4.0),
                     b=rng.uniform(20.0, 100.0), c=rng.uniform(0.02, 0.3))
    if path in ("reduce", "combine"):
        n = _logint(rng, 100, 20000)
        ops = ["mean", "sum", "std"] if path == "reduce" else ["sum", "sub", "sqdiff"]
        if dtype == "f32" or rng.random() < 0.25:
            # curves sampled at common times (the result's rows are then the
            # grid's, whatever the values)
            shape, lo = "grid", hi
            ops.append("max")
        else:
            shape = "walk"
        op = rng.choice(ops)
        group = _logint(rng, 2, 60) if op == "std" else _logint(rng, 2, n)
        return _case(path, n, lo, hi, dtype, shape=shape, op=op, group=group)
    return _case(path, _logint(rng, 200, 20000), lo, hi, dtype, p=rng.choice([1.0, 2.0, 3.0]))


# ---------------------------------------------------------------------------
# Inputs (host CSR arrays). A case fixes how many curves and rows there are,
# so that every seed gives results of one shape; times, values and loss
# weights come from the seed.

def _rng(*key):
    return np.random.Generator(np.random.PCG64(np.random.SeedSequence(key)))


def _curves(case, counts, seed, which):
    """Curves of ``counts`` rows: t_0 = 0, gaps 0.001 + 0.999 Exp(1) (so that
    times stay apart in single precision), last value 0. "walk": values N(0,1);
    "rank": nonincreasing integers from Poisson(50) down to 0; "grid": values
    N(0,1) at the common times 0, 1/8, 2/8, ..."""
    rng = _rng(seed, which)
    o = np.zeros(len(counts) + 1, dtype=np.int64)
    np.cumsum(counts, out=o[1:])
    k = np.arange(o[-1]) - np.repeat(o[:-1], counts)
    if case["shape"] == "grid":
        t = k / 8.0
    else:
        t = 1e-3 + 0.999 * rng.exponential(1.0, size=o[-1])
        t[o[:-1]] = 0.0
        for i in range(len(counts)):
            np.cumsum(t[o[i]:o[i + 1]], out=t[o[i]:o[i + 1]])
    if case["shape"] == "rank":
        top = np.repeat(rng.poisson(50.0, size=len(counts)), counts)
        e = np.cumsum(rng.exponential(1.0, size=o[-1]))
        s = e - np.repeat(e[o[:-1]], counts)
        end = np.repeat(s[o[1:] - 1], counts)
        v = np.floor((1.0 - s / np.maximum(end, 1e-12)) * top)
    else:
        v = rng.standard_normal(size=o[-1])
    v[o[1:] - 1] = 0.0
    dt = _DT[case["dtype"]]
    return o, t.astype(dt), v.astype(dt)


def _counts(case, n, which):
    return _rng(n, case["lo"], case["hi"], which).integers(case["lo"], case["hi"] + 1, size=n)


def _inputs(case, seed):
    path, n = case["path"], case["n"]
    if path == "batched":
        rng = _rng(n, case["smin"], case["smax"], case["mean"])
        sizes = np.rint(np.exp(rng.uniform(math.log(case["smin"]), math.log(case["smax"]),
                                           size=n))).astype(np.int64)
        so = np.append(0, np.cumsum(sizes))
        counts = np.minimum(rng.geometric(1.0 / case["mean"], size=so[-1]), case["hi"])
        return _curves(case, counts, seed, 0), so
    first = _curves(case, _counts(case, n, 0), seed, 0)
    if path == "cdist":
        return first, _curves(case, _counts(case, case["m"], 1), seed, 1)
    if path == "combine":
        return first, _curves(case, _counts(case, n, 1), seed, 1)
    if path == "grad":
        W = np.triu(_rng(seed, 2).uniform(0.0, 1.0, size=(n, n)))
        return first, W + np.triu(W, 1).T
    if path == "reduce":
        g = np.arange(0, n, case["group"], dtype=np.int64)
        if case["op"] == "std" and n - g[-1] < 2:
            g = g[:-1]  # a standard deviation needs two curves
        return first, np.append(g, n)
    return first, None


def prepare(case, seed):
    first, more = _inputs(case, seed)
    st = {"case": case, "X": api.PcfSet(*first)}
    path = case["path"]
    if path in ("cdist", "combine"):
        st["Y"] = api.PcfSet(*more)
    elif path == "batched":
        st["sets"] = more
    elif path == "reduce":
        st["groups"] = more
    elif path == "grad":
        X = st["X"]
        st["t"] = X.t.clone().requires_grad_(True)
        st["v"] = X.v.clone().requires_grad_(True)
        st["W"] = torch.as_tensor(more, device="cuda").to(X.dtype)
    return st


def _kind(case):
    if case["p"] == 0.0:
        return api.PCF_GRAM
    return api.PCF_LP_POW if case.get("power") else api.PCF_LP


def run(st):
    case, X = st["case"], st["X"]
    path, p = case["path"], case["p"]
    if path == "pdist":
        return api.gram(X) if p == 0.0 else api.pdist(X, p)
    if path == "window":
        return api.pdist(X, p, window=_window(case))
    if path == "cdist":
        return api.cross_gram(X, st["Y"]) if p == 0.0 else api.cdist(X, st["Y"], p)
    if path == "batched":
        return api.pairwise_batched(st["sets"], X, _kind(case), p)[0]
    if path == "grad":
        F = api.pairwise_matrix(X, st["t"], st["v"], _kind(case), p)
        gt, gv = torch.autograd.grad(F, (st["t"], st["v"]), grad_outputs=st["W"])
        return F.detach(), gt, gv
    if path == "ranged":
        return api.pdist(X, p, bounds=(case["a"], case["b"]), weight=("exp", case["c"]))
    if path == "reduce":
        R = api.reduce(X, case["op"], groups=st["groups"])
        return R.offsets, R.t, R.v
    if path == "combine":
        R = api.combine(X, st["Y"], case["op"])
        return R.offsets, R.t, R.v
    return api.norms(X, p)


def _window(case):
    """The last ``rows`` rows of the first quarter against every column after
    the first quarter: no pair lies in the window twice."""
    q = max(case["n"] // 4, case["rows"])
    return (q - case["rows"], q, q, case["n"])


# ---------------------------------------------------------------------------
# What a pass cannot do without

def _mean_rows(case):
    return case["mean"] if case["path"] == "batched" else 0.5 * (case["lo"] + case["hi"])


def work(case):
    path, n, e, r = case["path"], case["n"], _ESZ[case["dtype"]], _mean_rows(case)
    row = 2.0 * e  # a breakpoint's time and value
    # one merge step: compare, width, h, multiply-add
    ops = {0.0: 5.0, 1.0: 5.0, 2.0: 6.0}.get(case["p"], 12.0)
    if path == "pdist":
        return {"bytes": n * r * row + n * n * e, "flops": n * n / 2 * 2 * r * ops}
    if path == "window":
        r0, r1, c0, c1 = _window(case)
        k = (r1 - r0) * (c1 - c0)
        return {"bytes": (r1 - r0 + c1 - c0) * r * row + k * e, "flops": k * 2 * r * ops}
    if path == "cdist":
        k = n * case["m"]
        return {"bytes": (n + case["m"]) * r * row + k * e, "flops": k * 2 * r * ops}
    if path == "batched":
        # sizes are log-uniform: mean and mean square of exp(U(ln smin, ln smax))
        a, b = float(case["smin"]), float(max(case["smax"], case["smin"] + 1))
        s1, s2 = (b - a) / math.log(b / a), (b * b - a * a) / (2 * math.log(b / a))
        return {"bytes": n * (s1 * r * row + s2 * e), "flops": n * s2 / 2 * 2 * r * ops}
    if path == "grad":
        # forward and backward merges; loss weights, matrix and gradients once
        return {"bytes": 2 * n * r * row + 2 * n * n * e,
                "flops": n * n / 2 * 2 * r * (ops + 12.0)}
    if path == "ranged":
        kept = min(r, case["b"] - case["a"] + 2)
        return {"bytes": n * r * row + n * n * e, "flops": n * n / 2 * 2 * kept * ops}
    if path == "reduce":
        levels = math.ceil(math.log2(max(2, min(case["group"], n))))
        extra = 3.0 * case["group"] if case["op"] == "std" else 0.0
        return {"bytes": 2 * n * r * row, "flops": n * r * (2.0 * levels + extra)}
    if path == "combine":
        return {"bytes": 4 * n * r * row, "flops": 2 * n * r * 2.0}
    return {"bytes": n * r * row + n * (8 + e), "flops": n * r * 3.0}


# ---------------------------------------------------------------------------
# The same results in 64 bits (80 bits where NumPy's long double carries the
# sums), by evaluating both curves on the union of their breakpoints.

_MAX_ELEMENTS = 3.0e9  # union-grid elements that take a few seconds


def _pad(o, t, v, device):
    """Rows as dense arrays: times padded with the last time (cells of width
    0), values with the last value."""
    o = np.asarray(o)
    n, cnt = len(o) - 1, np.diff(o)
    idx = o[:-1, None] + np.minimum(np.arange(cnt.max())[None, :], cnt[:, None] - 1)
    return (torch.as_tensor(t.astype(np.float64)[idx], device=device),
            torch.as_tensor(v.astype(np.float64)[idx], device=device))


def _h(p, a, b):
    if p == 0.0:
        return a * b
    d = (a - b).abs()
    return d if p == 1.0 else (d * d if p == 2.0 else d ** p)


def _row(Ti, Vi, T, V, p, warp=None):
    """int h(f_i, f_j) for one curve i (rows Ti, Vi) and all curves j of T, V."""
    m, k = T.shape[0], Ti.shape[0]
    x, _ = torch.cat([Ti.expand(m, k), T], 1).sort(dim=1)
    key = x.detach().contiguous()
    ia = torch.searchsorted(Ti.detach().contiguous(), key, right=True) - 1
    ib = torch.searchsorted(T.detach().contiguous(), key, right=True) - 1
    h = _h(p, Vi[ia], V.gather(1, ib))
    w = (x if warp is None else warp(x)).diff(dim=1)
    return (h[:, :-1] * w).sum(1)


def _root(case, F):
    p = case["p"]
    return F if p in (0.0, 1.0) or case.get("power") else F ** (1.0 / p)


def _matrix(case, T, V, U, W, warp=None):
    return torch.stack([_root(case, _row(T[i], V[i], U, W, case["p"], warp))
                        for i in range(T.shape[0])])


def _elements(case, pairs, first):
    return pairs * 2.0 * float(np.diff(first[0]).max())


def exact(case, seed):
    path = case["path"]
    if path == "pdist" and case["n"] ** 2 * 2.0 * case["hi"] > _MAX_ELEMENTS:
        return None
    first, more = _inputs(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    o, t, v = first
    n = len(o) - 1
    if path in ("pdist", "window", "cdist", "ranged"):
        if path == "window":
            r0, r1, c0, c1 = _window(case)
        elif path == "cdist":
            r0, r1, c0, c1 = 0, n, 0, case["m"]
        else:
            r0, r1, c0, c1 = 0, n, 0, n
        if _elements(case, (r1 - r0) * (c1 - c0), first) > _MAX_ELEMENTS:
            return None
        T, V = _pad(o, t, v, dev)
        U, W = _pad(*more, dev) if path == "cdist" else (T, V)
        warp = None
        if path == "ranged":
            a, b, c = case["a"], case["b"], case["c"]
            if case["dtype"] == "f32":
                return None  # the warped times are rounded to the set's type
            # cells outside [a, b) get width 0
            warp = lambda x: -torch.expm1(-c * (x.clamp(a, b) - a)) * math.exp(-c * a) / c
        return _matrix(case, T[r0:r1], V[r0:r1], U[c0:c1], W[c0:c1], warp)
    if path == "batched":
        so, parts = more, []
        # (each problem padded to its own longest curve)
        size = np.diff(so)
        longest = np.maximum.reduceat(np.diff(o), so[:-1])
        if float((size.astype(np.float64) ** 2 * 2 * longest).sum()) > _MAX_ELEMENTS:
            return None
        for b in range(len(so) - 1):
            oo = o[so[b]:so[b + 1] + 1]
            T, V = _pad(oo - oo[0], t[oo[0]:oo[-1]], v[oo[0]:oo[-1]], dev)
            parts.append(_matrix(case, T, V, T, V).reshape(-1))
        return torch.cat(parts)
    if path == "grad":
        if _elements(case, n * n, first) > 1.5e9:
            return None
        T, V = _pad(o, t, v, dev)
        cnt = torch.as_tensor(np.diff(o), device=dev)
        k = torch.arange(T.shape[1], device=dev)[None, :]
        Wm = torch.as_tensor(more.astype(_DT[case["dtype"]]).astype(np.float64), device=dev)
        tf = torch.as_tensor(t.astype(np.float64), device=dev).requires_grad_(True)
        vf = torch.as_tensor(v.astype(np.float64), device=dev).requires_grad_(True)
        idx = torch.as_tensor(o[:-1], device=dev)[:, None] + torch.minimum(k, cnt[:, None] - 1)
        F = torch.zeros(n, n, dtype=torch.float64, device=dev)
        gt, gv = torch.zeros_like(tf), torch.zeros_like(vf)
        for i in range(n):
            # (a pair's padded cells have width 0, so nothing flows into them;
            # the padded times' own gradients cancel)
            sub = idx[i:]
            row = _row(tf[idx[i]], vf[idx[i]], tf[sub], vf[sub], case["p"])
            w = Wm[i, i:] + Wm[i:, i]
            w = torch.cat([w[:1] * 0.5, w[1:]])
            dF = torch.ones_like(row)
            r = row.detach()
            if case["p"] == 2.0 and not case.get("power"):
                dF = torch.where(r > 0, 0.5 / r.clamp_min(1e-300).sqrt(), torch.zeros_like(r))
            g = torch.autograd.grad(row, (tf, vf), grad_outputs=w * dF)
            gt += g[0]
            gv += g[1]
            F[i, i:] = F[i:, i] = _root(case, r)
        # a curve's first time and last value are fixed
        gt[torch.as_tensor(o[:-1], device=dev)] = 0.0
        gv[torch.as_tensor(o[1:] - 1, device=dev)] = 0.0
        return F, gt, gv
    ld = np.longdouble
    if path == "norms":
        w = np.append(np.diff(t.astype(ld)), 0)
        w[o[1:] - 1] = 0
        s = np.add.reduceat(np.abs(v.astype(ld)) ** int(case["p"]) * w, o[:-1])
        return (s ** (ld(1) / ld(case["p"]))).astype(np.float64)
    if path == "combine":
        return None  # every value is one rounded operation
    return _exact_reduce(case, o, t, v, more)


def _exact_reduce(case, o, t, v, groups):
    """Times and values of the reduced curves (sum, mean: running sums of the
    jumps in long double; std: every curve at every breakpoint)."""
    ld, op = np.longdouble, case["op"]
    if op == "max":
        return None  # no rounding
    offs, ts, vs = [0], [], []
    for b in range(len(groups) - 1):
        i0, i1 = groups[b], groups[b + 1]
        r0, r1 = o[i0], o[i1]
        x = np.unique(t[r0:r1])
        if i1 - i0 == 1:
            y = v[r0:r1].astype(ld)
            x = t[r0:r1]
        elif op == "std":
            at = np.stack([v[o[i]:o[i + 1]][np.searchsorted(t[o[i]:o[i + 1]], x, "right") - 1]
                           for i in range(i0, i1)]).astype(ld)
            d = at - at.mean(0)
            q = (d * d).sum(0)
            y = np.sqrt(q / ld(i1 - i0 - 1))
        else:
            jump = v[r0:r1].astype(ld)
            first = o[i0:i1] - r0
            prev = np.empty_like(jump)
            prev[1:] = jump[:-1]
            prev[first] = 0
            order = np.argsort(t[r0:r1], kind="stable")
            s = np.cumsum((jump - prev)[order])
            last = np.searchsorted(t[r0:r1][order], x, "right") - 1
            y = s[last]
            if op == "mean":
                y = y / ld(i1 - i0)
        offs.append(offs[-1] + len(x))
        ts.append(x)
        vs.append(np.asarray(y, dtype=np.float64))
    return None, np.concatenate(ts).astype(np.float64), np.concatenate(vs)
