"""Standard deviations of groups of at most 64 PCFs against the oracle, row for
row and bit for bit: group sizes around the four values that are summed
together, and times on a coarse grid, so that runs of equal times (up to the
whole group) end inside a block of 64 rows, at its end, past it, and at the end
of a chunk of 1,024 rows.
"""
import numpy as np
import pytest

from oracle import reduce as red
from paper_2404_07183_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("keep", [0.05, 0.5, 1.0])
@pytest.mark.parametrize("m", [2, 3, 4, 5, 7, 20, 33, 63, 64])
def test_std_rows(m, keep, dtype):
    # every PCF keeps each dyadic grid time with probability `keep`
    rng = np.random.default_rng(m)
    grid = np.arange(1, 1 + int(np.ceil(2600 / (m * keep))))
    ts, vs, o = [], [], [0]
    groups = [0, m, 2 * m, 2 * m + 2]
    for _ in range(groups[-1]):
        t = np.concatenate([[0], grid[rng.random(len(grid)) < keep]]) / 8.0
        v = rng.standard_normal(len(t))
        v[-1] = 0
        ts.append(t)
        vs.append(v)
        o.append(o[-1] + len(t))
    o = np.array(o)
    t, v = np.concatenate(ts).astype(dtype), np.concatenate(vs).astype(dtype)
    R = api.reduce(api.PcfSet(o, t, v, device="cuda:0"), "std", groups)
    oo, tt, vv = R.offsets_host, R.t.cpu().numpy(), R.v.cpu().numpy()
    for b, (wt, wv) in enumerate(red.reduce_groups("std", groups, o, t, v, dtype=dtype)):
        assert np.array_equal(tt[oo[b]:oo[b + 1]], wt), b
        assert np.array_equal(vv[oo[b]:oo[b + 1]], wv), b
