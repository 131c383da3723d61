"""The strip kernel through the calls that reach it beside the plain matrix, in
both types, against the CPU oracle: sums of terms (each term after the first is
added to the entries the first one wrote), batches, ranges and time weights.

Bars: FP64 1e-12, FP32 1e-5 of the magnitudes of the terms that make up an entry
(sum over its cells of |h0| (|W(r)| + |W(l)|), times |coefficient|).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_07183_amd import api, workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BAR = {np.float64: 1e-12, np.float32: 1e-5}
TERMS = [("lp", 1.0, None, 1.0), ("gram", 0.0, ("exp", 0.5), -0.7), ("lp", 3.0, ("pow", 0.5), 0.2)]
N = 2003


def _is_strip(ws):
    return int(ws.buf[192:196].view(torch.int32)[0]) > 0


def _set(dtype, n=N, seed=31):
    return workloads.uniform_counts(n, 5, 60, seed=seed, dtype=dtype)


def _terms(o, t, v, I, J):
    """The sum and the magnitudes of its parts."""
    s, ab = np.zeros(len(I)), np.zeros(len(I))
    for h0, p, w, coef in TERMS:
        kind = oracle.LP_POW if h0 == "lp" else oracle.GRAM
        if w is None:
            r, a = oracle.entries(kind, p, o, t, v, I, J, with_abs=True)
        else:
            r, a = oracle.entries_w(kind, p, oracle.W_EXP if w[0] == "exp" else oracle.W_POW, w[1],
                                    o, t, v, I, J, with_abs=True)
        s += coef * r
        ab += abs(coef) * a
    return s, ab


def _sample(r0, r1, c0, c1, count=20000, seed=6):
    rng = np.random.default_rng(seed)
    k = min(r1 - r0, c1 - c0, 300)
    return (np.concatenate([rng.integers(r0, r1, size=count), r0 + np.arange(k)]),
            np.concatenate([rng.integers(c0, c1, size=count), c0 + np.arange(k)]))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("window", [None, (100, 1500, 300, 2003), (0, 2003, 40, 1500)])
def test_terms(dtype, window):
    o, t, v = _set(dtype)
    X = api.PcfSet(o, t, v, device=DEV)
    ws = api.Workspace()
    w = window or (0, N, 0, N)
    M = api.pairwise_terms(X, TERMS, window=window, workspace=ws).cpu().numpy()
    assert _is_strip(ws)
    I, J = _sample(*w)
    ref, ab = _terms(o, t, v, I, J)
    assert np.all(np.abs(M[I - w[0], J - w[2]] - ref) <= BAR[dtype] * ab)
    if window is None:
        assert np.array_equal(M, M.T)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_terms_upper_only(dtype):
    o, t, v = _set(dtype)
    X = api.PcfSet(o, t, v, device=DEV)
    out = torch.full((N, N + 2), 7.0, dtype=X.dtype, device=DEV)
    ws = api.Workspace()
    api.pairwise_terms(X, TERMS, out=out, upper_only=True, workspace=ws)
    assert _is_strip(ws)
    up, full = out.cpu().numpy(), api.pairwise_terms(X, TERMS).cpu().numpy()
    iu = np.triu_indices(N)
    assert np.array_equal(up[:, :N][iu], full[iu])
    assert np.all(up[:, :N][np.tril_indices(N, -1)] == 7.0) and np.all(up[:, N:] == 7.0)


@pytest.mark.parametrize("kind,p", [(api.PCF_LP, 1.0), (api.PCF_LP, 3.5), (api.PCF_GRAM, 0.0)])
def test_batched_fp32(kind, p):
    sizes = np.array([1, 900, 64, 65, 1700, 3, 1601])
    so = np.concatenate([[0], np.cumsum(sizes)])
    o, t, v = _set(np.float32, int(so[-1]), 32)
    X = api.PcfSet(o, t, v, device=DEV)
    ws = api.Workspace()
    out, oo = api.pairwise_batched(so, X, kind, p, workspace=ws)
    assert _is_strip(ws)
    out = out.cpu().numpy()
    for b, s in enumerate(sizes):
        I, J = _sample(0, s, 0, s, 3000)
        ref, ab = oracle.entries(kind, p, o, t, v, so[b] + I, so[b] + J, with_abs=True)
        sc = ab ** (1.0 / p) if kind == api.PCF_LP else ab
        got = out[oo[b]:oo[b] + s * s].reshape(s, s)[I, J]
        assert np.all(np.abs(got - ref) <= 1e-5 * np.maximum(sc, 1e-30)), b


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("kind", ["l1", "gram"])
def test_range_and_weight(dtype, kind):
    o, t, v = _set(dtype)
    X = api.PcfSet(o, t, v, device=DEV)
    ws = api.Workspace()
    a, b, c = 0.5, 20.0, 0.125  # (exact in both types)
    fn = (lambda **k: api.pdist(X, 1.0, **k)) if kind == "l1" else (lambda **k: api.gram(X, **k))
    M = fn(bounds=(a, b), weight=("exp", c), workspace=ws).cpu().numpy()
    assert _is_strip(ws)
    I, J = _sample(0, N, 0, N)
    ref, ab = oracle.entries_w(oracle.LP if kind == "l1" else oracle.GRAM, 1.0, oracle.W_EXP, c, o,
                               t, v, I, J, a=a, b=b, with_abs=True)
    assert np.all(np.abs(M[I, J] - ref) <= BAR[dtype] * ab)
