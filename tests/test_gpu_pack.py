"""The packed breakpoint records in the workspace, bit for bit against records
made with numpy: sets on both sides of each rule that chooses the packing
kernel (16 lanes a PCF, a wave a PCF, a wave for a run of rows whatever their
PCFs), row counts around the runs' length, and sets of one to many thousand
PCFs around a long one (one to three rounds of the search for a run's PCF)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2404_07183_amd import _lib, api

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
PAD = 7
OFF_REC = 32 + 6 * 8  # of the workspace header: counters, four counts, two offsets

COUNTS = {
    "one row": [1],
    "16 lanes": [3, 20, 1, 25] * 40,
    "16 lanes' longest": [5] * 60 + [256],
    "a wave": [5] * 60 + [257],
    "a wave's longest": [60, 1999, 1, 64],
    "rows": [60, 2000, 1, 64],
    "rows alone": [2000],
    "runs of 512": [512, 2048, 511, 1, 513, 1, 1, 1, 509, 2049, 3],
    "one-row PCFs around": [1] * 700 + [2100] + [1] * 700 + [5000] + [1] * 65,
    "search of two rounds": [2] * 64 + [3000] + [1] * 4000,
    "search of three rounds": [3] * 4096 + [2500] + [7] * 3000 + [1],
    "very long": [1, 100003, 2, 60000, 30],
    "longer runs": [700001, 64, 128, 1, 420000, 127, 65],
}


def _set(counts, dtype, seed=1):
    o = np.concatenate([[0], np.cumsum(counts)])
    t = (np.arange(o[-1]) - np.repeat(o[:-1], counts)) / 4.0
    v = np.random.default_rng(seed).standard_normal(o[-1])
    v[o[1:] - 1] = 0.0
    return o, t.astype(dtype), v.astype(dtype)


def _records(o, t, v):
    """Per row (end of its piece, value), the last row PAD more times, each
    PCF's last piece ending at the sentinel (read from the result)."""
    end, val = [], []
    for a, b in zip(o[:-1], o[1:]):
        end += [t[a + 1:b], np.full(1 + PAD, np.inf, t.dtype)]
        val += [v[a:b], np.full(PAD, v[b - 1])]
    return np.concatenate(end), np.concatenate(val)


def _check(ws, o, t, v):
    buf = ws.buf.cpu().numpy()
    at = int(buf[OFF_REC:OFF_REC + 8].view(np.int64)[0])
    n = int(o[-1]) + PAD * (len(o) - 1)
    rec = buf[at:at + n * 2 * t.itemsize].view(t.dtype).reshape(n, 2)
    end, val = _records(o, t, v)
    last = np.isinf(end)
    assert np.array_equal(rec[~last, 0], end[~last])
    assert np.all(rec[last, 0] == rec[last, 0][0]) and rec[last, 0][0] > 1e30
    assert np.array_equal(rec[:, 1], val)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("name", list(COUNTS))
def test_records(name, dtype):
    o, t, v = _set(COUNTS[name], dtype)
    X = api.PcfSet(o, t, v, device=DEV)
    n = X.n
    window = (0, min(n, 2), max(0, n - 2), n)  # (the whole set is packed)
    ws = api.Workspace()
    api.pdist(X, 1.0, window=window, workspace=ws)
    _check(ws, o, t, v)
    # new data through the same plan, by a caller without host offsets
    o, t2, v2 = _set(COUNTS[name], dtype, seed=2)
    Y = api.PcfSet(o, t2, v2, device=DEV)
    c = Y.c_struct()
    c.offsets_host = None
    out = torch.empty((window[1], n - window[2]), dtype=Y.dtype, device=DEV)
    _lib.check(_lib.pcf_pairwise_lp(c, api.PCF_LP, 1.0, out.data_ptr(), out.shape[1],
                                    api._window(window), ws.ptr, ws.nbytes,
                                    api.PCF_REUSE_PLAN, api._stream_handle()))
    _check(ws, o, t2, v2)


@pytest.mark.parametrize("a,b", [("16 lanes", "rows"), ("runs of 512", "16 lanes"),
                                 ("rows", "runs of 512")])
def test_cross_records(a, b):
    oa, ta, va = _set(COUNTS[a], np.float64, 3)
    ob, tb, vb = _set(COUNTS[b], np.float64, 4)
    ws = api.Workspace()
    api.cdist(api.PcfSet(oa, ta, va, device=DEV), api.PcfSet(ob, tb, vb, device=DEV), 1.0,
              workspace=ws)
    _check(ws, np.concatenate([oa, oa[-1] + ob[1:]]), np.concatenate([ta, tb]),
           np.concatenate([va, vb]))
