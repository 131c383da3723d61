"""The strip kernel on sets of very uneven lengths, against the CPU oracle: row
blocks kept small because a long column would outlast the launch (several columns
an item), the longest PCF limiting the columns an item has, long PCFs on the
resident and on the streamed side, and sets that the rule leaves to tiles.

Bars as in test_gpu_strips.py: FP64 1e-12, FP32 1e-5 of the entry's scale.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_07183_amd import api, workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = {np.float64: 1e-12, np.float32: 1e-5}


def _set(n, rows, longs, seed, dtype):
    """n PCFs of `rows` rows, of `longs` = {index: rows}."""
    rng = np.random.default_rng(seed)
    c = np.full(n, rows)
    for i, r in longs.items():
        c[i] = r
    o = np.concatenate([[0], np.cumsum(c)])
    s = np.cumsum(np.where(np.isin(np.arange(o[-1]), o[:-1]), 0.0, rng.exponential(1.0, o[-1])))
    t = s - np.repeat(s[o[:-1]], c)
    v = rng.standard_normal(o[-1])
    v[o[1:] - 1] = 0.0
    return workloads.to_dtype(o, t, v, dtype)


def _plan(ws):
    """Rows a block (0: a tile plan) and columns an item, of a strip plan."""
    pairs, cols = (int(x) for x in ws.buf[192:200].view(torch.int32))
    return (pairs // cols, cols) if pairs > 0 else (0, 0)


def _check(M, o, t, v, p, r0, r1, c0, c1, tol, extra=(), samples=40000):
    """Sampled entries and every entry of rows and columns `extra`."""
    rng = np.random.default_rng(5)
    I, J = [rng.integers(r0, r1, size=samples)], [rng.integers(c0, c1, size=samples)]
    for e in extra:
        if r0 <= e < r1:
            I.append(np.full(c1 - c0, e))
            J.append(np.arange(c0, c1))
        if c0 <= e < c1:
            I.append(np.arange(r0, r1))
            J.append(np.full(r1 - r0, e))
    I, J = np.concatenate(I), np.concatenate(J)
    ref, ab = oracle.entries(oracle.LP, p, o, t, v, I, J, with_abs=True)
    err = np.abs(M[I - r0, J - c0].astype(np.float64) - ref)
    assert np.all(err <= tol * np.maximum(ab ** (1.0 / p), 1e-300)), err.max()


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n,rows,every,long", [(2000, 30, 100, 600), (2000, 20, 25, 300),
                                               (2003, 30, 450, 900)])
def test_small_blocks(n, rows, every, long, dtype):
    longs = {i: long for i in range(every // 2, n, every)}
    o, t, v = _set(n, rows, longs, 21, dtype)
    X = api.PcfSet(o, t, v, device=DEV)
    ws = api.Workspace()
    M = api.pdist(X, 1.0, workspace=ws).cpu().numpy()
    R, C = _plan(ws)
    assert 12 <= R < 64 and C > 1
    _check(M, o, t, v, 1.0, 0, n, 0, n, TOL[dtype], list(longs)[:3] + list(longs)[-2:])
    assert np.array_equal(M, M.T)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_longest_limits_the_columns(dtype):
    n, longs = 7000, {5: 3000, 1757: 3000, 3507: 2990, 6999: 3000}
    o, t, v = _set(n, 40, longs, 22, dtype)
    X = api.PcfSet(o, t, v, device=DEV)
    ws = api.Workspace()
    M = api.pdist(X, 2.0, workspace=ws).cpu().numpy()
    R, C = _plan(ws)
    assert R == 64 and C >= 2
    _check(M, o, t, v, 2.0, 0, n, 0, n, TOL[dtype], list(longs), samples=20000)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("window", [(100, 1900, 900, 2600), (3, 1203, 600, 2600),
                                    (0, 2600, 40, 1240)])
def test_windows(window, dtype):
    longs = {150: 700, 950: 700, 1500: 650, 2550: 700}
    o, t, v = _set(2600, 40, longs, 23, dtype)
    X = api.PcfSet(o, t, v, device=DEV)
    ws = api.Workspace()
    M = api.pdist(X, 1.0, window=window, workspace=ws).cpu().numpy()
    assert _plan(ws)[0] > 0
    _check(M, o, t, v, 1.0, *window, TOL[dtype], longs)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("longs_x,longs_y", [({7: 800, 300: 800}, {}), ({}, {9: 800, 3000: 780})])
def test_cross(longs_x, longs_y, dtype):
    # long PCFs among the resident rows (X, the short side), then among the columns
    a, b = _set(900, 30, longs_x, 24, dtype), _set(4500, 30, longs_y, 25, dtype)
    X, Y = api.PcfSet(*a, device=DEV), api.PcfSet(*b, device=DEV)
    ws = api.Workspace()
    M = api.cdist(X, Y, 1.0, workspace=ws).cpu().numpy()
    assert _plan(ws)[0] > 0
    o = np.concatenate([a[0], a[0][-1] + b[0][1:]])
    t, v = np.concatenate([a[1], b[1]]), np.concatenate([a[2], b[2]])
    _check(M, o, t, v, 1.0, 0, 900, 900, 5400, TOL[dtype],
           list(longs_x) + [900 + k for k in longs_y])


@pytest.mark.parametrize("n,rows,longs", [(1800, 40, {400: 3000, 900: 3000, 1700: 3000}),
                                          (2500, 20, {k: 2500 for k in range(50, 2500, 100)}),
                                          (2500, 100, {k: 400 for k in range(5, 2500, 10)})])
def test_left_to_tiles(n, rows, longs):
    o, t, v = _set(n, rows, longs, 26, np.float64)
    X = api.PcfSet(o, t, v, device=DEV)
    ws = api.Workspace()
    M = api.pdist(X, 1.0, workspace=ws).cpu().numpy()
    assert _plan(ws) == (0, 0)
    _check(M, o, t, v, 1.0, 0, n, 0, n, 1e-12, list(longs)[:2])
