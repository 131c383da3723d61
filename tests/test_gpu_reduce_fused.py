"""Reduction passes over several tree levels at once, against the oracle's
ReducePair tree, row for row and bit for bit: group sizes around the 16 items
of a bundle and the passes' level counts, PCFs on both sides of the samples'
spacing (48 rows) and long ones (many tiles a bundle), and common time grids
(every breakpoint shared by all PCFs, so that tiles split runs of equal times).
"""
import numpy as np
import pytest

from oracle import reduce as red
from paper_2404_07183_amd import api, workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(o, t, v, groups, op, dtype=np.float64):
    X = api.PcfSet(o, t, v, device=DEV)
    R = api.reduce(X, op, groups)
    oo, tt, vv = R.offsets_host, R.t.cpu().numpy(), R.v.cpu().numpy()
    want = red.reduce_groups(op, groups, o, t, v, dtype=dtype)
    assert np.array_equal(R.offsets.cpu().numpy(), oo)
    for b, (wt, wv) in enumerate(want):
        assert np.array_equal(tt[oo[b]:oo[b + 1]], wt), (op, b)
        assert np.array_equal(vv[oo[b]:oo[b + 1]], wv), (op, b)


@pytest.mark.parametrize("m", [2, 3, 4, 15, 16, 17, 31, 32, 33, 64, 65, 257])
@pytest.mark.parametrize("op", ["sum", "max"])
def test_group_sizes(m, op):
    # three groups of m and one of a single PCF: unpaired items at every level
    o, t, v = workloads.uniform_counts(3 * m + 1, 1, 60, seed=300 + m)
    _check(o, t, v, [0, m, 2 * m, 3 * m, 3 * m + 1], op)


@pytest.mark.parametrize("lo,hi", [(47, 49), (95, 97), (1, 1), (1, 4), (2000, 2600)])
def test_rows_around_the_spacing(lo, hi):
    o, t, v = workloads.uniform_counts(20, lo, hi, seed=400 + lo)
    _check(o, t, v, [0, 20], "sum")
    _check(o, t, v, [0, 5, 20], "min")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("rows", [3, 50, 400])
def test_common_grid(dtype, rows):
    # dyadic times shared by all PCFs: runs of 40 equal times across tiles
    n = 40
    rng = np.random.default_rng(rows)
    o = np.arange(n + 1) * rows
    t = np.tile(np.arange(rows) / 8.0, n).astype(dtype)
    v = rng.standard_normal(n * rows).astype(dtype)
    v[o[1:] - 1] = 0
    for op in ("sum", "max"):
        _check(o, t, v, [0, n], op, dtype)
    _check(o, t, v, [0, 3, n], "min", dtype)


def test_std_over_fused_passes_and_empty_call():
    o, t, v = workloads.uniform_counts(150, 2, 90, seed=500)
    _check(o, t, v, [0, 20, 63, 127, 150], "std")
    X = api.PcfSet(np.array([0]), np.zeros(0), np.zeros(0), device=DEV)
    assert api.reduce(X, "sum", groups=[0]).n == 0
