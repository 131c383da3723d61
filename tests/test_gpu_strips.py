"""The strip kernel (row blocks resident in LDS, columns streamed through it)
against the CPU oracle, at the sets and windows that select it: short PCFs in
large numbers, so that an item has several columns, row blocks of 64, one-row
and very long PCFs among them.

Bars: FP64 |gpu - oracle| <= 1e-12 * scale per entry, FP32 1e-5 * scale
against the oracle on the rounded inputs (scale: sum |h| * width, to the
power 1/p for d_p).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_07183_amd import _lib, api, workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _set(n, seed, dtype=np.float64, mean=30, longest=900):
    """Geometric row counts (one-row PCFs among them) and a few long PCFs."""
    rng = np.random.default_rng(seed)
    counts = np.minimum(rng.geometric(1.0 / mean, size=n), 6 * mean)
    counts[rng.integers(0, n, size=4)] = longest
    o = np.concatenate([[0], np.cumsum(counts)])
    t = rng.exponential(1.0, o[-1])
    t[o[:-1]] = 0.0
    for i in range(n):
        np.cumsum(t[o[i]:o[i + 1]], out=t[o[i]:o[i + 1]])
    v = rng.standard_normal(o[-1])
    v[o[1:] - 1] = 0.0
    return workloads.to_dtype(o, t, v, dtype)


def _is_strip(ws):
    """Whether a workspace holds a strip plan (strip_pairs of its header)."""
    return int(ws.buf[192:196].view(torch.int32)[0]) > 0


def _check(M, o, t, v, okind, p, r0, r1, c0, c1, tol, samples=60000, seed=3):
    rng = np.random.default_rng(seed)
    I = rng.integers(r0, r1, size=samples)
    J = rng.integers(c0, c1, size=samples)
    k = min(r1 - r0, c1 - c0, 500)  # the corner's diagonal band too
    I = np.concatenate([I, r0 + np.arange(k)])
    J = np.concatenate([J, c0 + np.arange(k)])
    ref, ab = oracle.entries(okind, p, o, t, v, I, J, with_abs=True)
    sc = ab ** (1.0 / p) if okind == oracle.LP and p != 1.0 else ab
    got = M[I - r0, J - c0].astype(np.float64)
    err = np.abs(got - ref)
    bad = err > tol * np.maximum(sc, 1e-300)
    assert not bad.any(), (np.argwhere(bad)[:5], err[bad][:5], ref[bad][:5])


CALLS = {"l1": (lambda X, **k: api.pdist(X, 1.0, **k), oracle.LP, 1.0),
         "l2": (lambda X, **k: api.pdist(X, 2.0, **k), oracle.LP, 2.0),
         "gram": (lambda X, **k: api.gram(X, **k), oracle.GRAM, 0.0),
         "l3.5": (lambda X, **k: api.pdist(X, 3.5, **k), oracle.LP, 3.5),
         "l2.7": (lambda X, **k: api.pdist(X, 2.7, **k), oracle.LP, 2.7)}


@pytest.mark.parametrize("name", sorted(CALLS))
@pytest.mark.parametrize("dtype,tol", [(np.float64, 1e-12), (np.float32, 1e-5)])
@pytest.mark.parametrize("mean", [3, 30])
def test_full_matrix(name, dtype, tol, mean):
    n = 2003 if mean == 30 else 5001
    o, t, v = _set(n, 11, dtype, mean)
    X = api.PcfSet(o, t, v, device=DEV)
    fn, okind, p = CALLS[name]
    ws = api.Workspace()
    M = fn(X, workspace=ws).cpu().numpy()
    assert _is_strip(ws)
    _check(M, o, t, v, okind, p, 0, n, 0, n, tol)
    assert np.array_equal(M, M.T)
    if name != "gram":
        assert np.all(np.diag(M) == 0)
    # only the upper triangle, into a wider matrix
    out = torch.full((n, n + 3), 7.0, dtype=X.dtype, device=DEV)
    fn(X, out=out, upper_only=True)
    up = out.cpu().numpy()
    il = np.tril_indices(n, -1)
    assert np.all(up[il] == 7.0) and np.all(up[:, n:] == 7.0)
    iu = np.triu_indices(n)
    assert np.array_equal(up[iu], M[iu])


@pytest.mark.parametrize("window", [(100, 1900, 900, 2600), (0, 2600, 40, 1240),
                                    (3, 1203, 600, 2600), (500, 2500, 500, 2500)])
def test_windows(window):
    # overlapping parts, a tall window (columns resident, rows streamed), a
    # wide one, a symmetric one
    n = 2600
    o, t, v = _set(n, 12, mean=60, longest=1500)
    X = api.PcfSet(o, t, v, device=DEV)
    ws = api.Workspace()
    M = api.pdist(X, 1.0, window=window, workspace=ws).cpu().numpy()
    assert _is_strip(ws)
    _check(M, o, t, v, oracle.LP, 1.0, *window, 1e-12)


def test_cross_tall_and_wide():
    a, b = _set(4100, 13), _set(801, 14)
    X, Y = api.PcfSet(*a, device=DEV), api.PcfSet(*b, device=DEV)
    ws = api.Workspace()
    M = api.cdist(X, Y, 1.0, workspace=ws).cpu().numpy()
    assert _is_strip(ws)
    W = api.cdist(Y, X, 1.0).cpu().numpy()
    o = np.concatenate([a[0], a[0][-1] + b[0][1:]])
    t, v = np.concatenate([a[1], b[1]]), np.concatenate([a[2], b[2]])
    _check(M, o, t, v, oracle.LP, 1.0, 0, 4100, 4100, 4901, 1e-12)
    assert np.max(np.abs(M - W.T)) <= 1e-12 * max(1.0, np.max(M))


def test_long_pcfs_few_waves():
    # PCFs of hundreds of rows: fewer waves a workgroup, columns longer than
    # the registers that a wave loads ahead
    o, t, v = workloads.uniform_counts(700, 300, 1500, seed=15)
    X = api.PcfSet(o, t, v, device=DEV)
    ws = api.Workspace()
    M = api.pdist(X, 2.0, workspace=ws).cpu().numpy()
    assert _is_strip(ws)
    _check(M, o, t, v, oracle.LP, 2.0, 0, 700, 0, 700, 1e-12, samples=4000)
    assert np.array_equal(M, M.T)


def test_batched_strips():
    rng = np.random.default_rng(16)
    sizes = np.array([0, 1, 2, 700, 65, 64, 63, 1700, 1, 3, 1601, 130])
    o, t, v = _set(int(sizes.sum()), 17)
    so = np.concatenate([[0], np.cumsum(sizes)])
    X = api.PcfSet(o, t, v, device=DEV)
    ws = api.Workspace()
    out, oo = api.pairwise_batched(so, X, api.PCF_LP, 1.0, workspace=ws)
    assert _is_strip(ws)
    out = out.cpu().numpy()
    for b, s in enumerate(sizes):
        if s == 0:
            continue
        a = so[b]
        M = out[oo[b]:oo[b] + s * s].reshape(s, s)
        o2 = o[a:a + s + 1] - o[a]
        _check(M, o2, t[o[a]:o[a + s]], v[o[a]:o[a + s]], oracle.LP, 1.0, 0, s, 0, s, 1e-12,
               samples=3000)


def test_reused_plan_new_data_and_p():
    o, t, v = _set(2003, 18)
    X = api.PcfSet(o, t, v, device=DEV)
    ws = api.Workspace()
    A = api.pdist(X, 1.0, workspace=ws)
    assert _is_strip(ws)
    Y = X.with_values(X.t, -2.0 * X.v)
    B = api.pdist(Y, 1.0, workspace=ws)
    assert torch.equal(B, 2.0 * A)
    C = api.pdist(X, 3.0, workspace=ws).cpu().numpy()  # another kernel, the same plan
    _check(C, o, t, v, oracle.LP, 3.0, 0, 2003, 0, 2003, 1e-12)


def test_workspace_of_the_tile_plan():
    # a workspace sized for the tile plan alone still serves the call
    n = 2003
    o, t, v = _set(n, 19)
    X = api.PcfSet(o, t, v, device=DEV)

    def up(x):
        return (x + 255) // 256 * 256
    nbytes = 256 + up((n + 1) * 4) + up(80) + up((int(o[-1]) + 7 * n) * 16)
    assert nbytes < _lib.pcf_workspace_bytes(X.c_struct(), api.PCF_LP, None, 0)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    out = torch.empty((n, n), dtype=torch.float64, device=DEV)
    _lib.check(_lib.pcf_pairwise_lp(X.c_struct(), api.PCF_LP, 1.0, out.data_ptr(), n, None,
                                    ws.data_ptr(), nbytes, 0, api._stream_handle()))
    _check(out.cpu().numpy(), o, t, v, oracle.LP, 1.0, 0, n, 0, n, 1e-12)
