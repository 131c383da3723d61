"""The fused reduction pass on the fullest tiles that sampling can give, against
the oracle's ReducePair tree, bit for bit.

A tile starts at every kFuseRanks-th sample of a bundle's 16 items (each item is
sampled every kFuseSpacing rows). It is fullest when, at its start, every item
but the starting one has just passed a sample and, at its end, all but one lie
just before their next one: kFuseRanks * kFuseSpacing + 15 (kFuseSpacing - 1)
rows, against kFuseRanks * kFuseSpacing on average. The layout below builds such
a tile as the bundle's second one; its row count is worked out here from the
kernel's constants and the sampling rule, so that the case stays at the bound.
"""
import os
import re

import numpy as np
import pytest

from oracle import reduce as red
from paper_2404_07183_amd import api

CSRC = os.path.join(os.path.dirname(api.__file__), "csrc")


def _constants():
    with open(os.path.join(CSRC, "reduce.hpp")) as f:
        h = f.read()
    with open(os.path.join(CSRC, "reduce.hip")) as f:
        k = f.read()
    levels, spacing, ranks = (int(re.search(r"constexpr int %s = (\d+);" % n, h).group(1))
                              for n in ("kFuseLevels", "kFuseSpacing", "kFuseRanks"))
    threads = int(re.search(r"constexpr int kFuseThreads = (\d+);", k).group(1))
    return 1 << levels, spacing, ranks, threads


def _full_tile_set(seed, dtype, fewer=0):
    """One bundle whose second tile is the fullest (``fewer``: rows left out of
    it); times are places in the merged order, exact in either dtype."""
    items, S, ranks, _ = _constants()
    rng = np.random.default_rng(seed)
    order = []  # the item of every row after the items' rows at time 0
    rows = np.ones(items, dtype=int)

    def burst(i, n):
        order.extend([i] * n)
        rows[i] += n

    # samples up to the tile's start: items 0, 1, .. in turn, to a sample each
    i = 0
    for _ in range(ranks - items):
        burst(i, S - (rows[i] - 1) % S)
        i = (i + 1) % items
    burst(0, S - (rows[0] - 1) % S)  # the tile's first row, item 0's sample
    start = len(order) - 1
    # its other samples go to the other items in turn; every item then runs on
    # to the row before its next sample
    extra = np.zeros(items, dtype=int)
    for u in range(ranks - 1):
        extra[1 + u % (items - 1)] += 1
    tile = []
    for j in range(items):
        n = S * extra[j] + S - 1 - (rows[j] - 1) % S
        tile += [j] * n
        rows[j] += n
    tile = list(rng.permutation(tile))
    for j in tile[:fewer]:
        rows[j] -= 1
    order += tile[fewer:]
    # past its end: item 0's next sample first, then a few rows of each
    for j in range(items):
        burst(j, 1 + j % 3)
    perm = rng.permutation(items)
    perm[np.argwhere(perm == 0)[0, 0]], perm[0] = perm[0], 0  # (item 0 starts the ties)
    t = [[0.0] for _ in range(items)]
    for k, j in enumerate(order):
        t[perm[j]].append(float(k + 1))
    o = np.concatenate([[0], np.cumsum([len(x) for x in t])])
    v = rng.standard_normal(o[-1])
    v[o[1:] - 1] = 0.0
    return o, np.concatenate(t).astype(dtype), v.astype(dtype), start


def _tile_rows(o, t):
    """Rows of each tile of one bundle by the sampling rule."""
    items, S, ranks, _ = _constants()
    item = np.repeat(np.arange(items), np.diff(o))
    index = np.arange(o[-1]) - o[item]
    sel = np.lexsort((index, item, t))
    sample = index[sel] % S == 0
    starts = np.flatnonzero(sample)[::ranks]
    return np.diff(np.concatenate([starts, [len(sel)]]))


def test_layout_fills_a_tile():
    items, S, ranks, threads = _constants()
    o, t, v, _ = _full_tile_set(1, np.float64)
    most = ranks * S + (items - 1) * (S - 1)
    rows = _tile_rows(o, t)
    assert rows[1] == most and rows.max() == most
    # a thread of the kernel takes ceil(rows / threads) of them in one run
    assert most > (most // threads) * threads


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("op", ["sum", "max", "std"])
def test_full_tiles(op, dtype):
    parts = [_full_tile_set(seed, dtype, fewer) for seed, fewer in ((1, 0), (2, 64), (3, 65), (4, 0))]
    n = len(parts[0][0]) - 1
    o = np.concatenate([[0]] + [p[0][1:] + sum(q[0][-1] for q in parts[:k])
                                for k, p in enumerate(parts)])
    t, v = np.concatenate([p[1] for p in parts]), np.concatenate([p[2] for p in parts])
    groups = [n * k for k in range(len(parts) + 1)]
    R = api.reduce(api.PcfSet(o, t, v, device="cuda:0"), op, groups)
    oo, tt, vv = R.offsets_host, R.t.cpu().numpy(), R.v.cpu().numpy()
    for b, (wt, wv) in enumerate(red.reduce_groups(op, groups, o, t, v, dtype=dtype)):
        assert np.array_equal(tt[oo[b]:oo[b + 1]], wt), (op, b)
        assert np.array_equal(vv[oo[b]:oo[b + 1]], wv), (op, b)
