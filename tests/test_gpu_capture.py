"""Calls under stream capture. A call that would make a plan is refused (the
plan would not be in the workspace before the graph's first replay), whatever
its plan's size, and the workspace serves eager calls as before; a call that
reuses a plan is captured, and every replay equals the eager result."""
import gc

import numpy as np
import pytest
import torch

from paper_2404_07183_amd import _lib, api, workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# plans of one kernel argument, of three, and by copy (a tile and a strip plan)
SETS = [(40, 5, 40), (1001, 10, 100), (700, 300, 1500), (2003, 5, 80)]


def _capture(fn):
    """Runs fn on a capturing stream; returns the graph (never empty). No garbage
    collection meanwhile: an older graph that it freed would synchronise the
    device, which a capture does not allow (an exception in its destructor)."""
    g, s, x = torch.cuda.CUDAGraph(), torch.cuda.Stream(), torch.zeros(8, device=DEV)
    s.wait_stream(torch.cuda.current_stream())
    gc.collect()
    gc.disable()
    try:
        with torch.cuda.stream(s):
            with torch.cuda.graph(g, stream=s):
                x.add_(1.0)
                fn()
    finally:
        gc.enable()
    torch.cuda.current_stream().wait_stream(s)
    return g


def _refused(call):
    got = []

    def fn():
        try:
            call()
            got.append(_lib.PCF_OK)
        except _lib.PcfError as e:
            got.append(e.status)  # (the exception itself would keep the graph alive)
    _capture(fn)
    assert got == [_lib.PCF_EDEVICE]


@pytest.mark.parametrize("n,lo,hi", SETS)
def test_new_plans_are_refused_and_reused_ones_replay(n, lo, hi):
    o, t, v = workloads.uniform_counts(n, lo, hi, seed=n)
    X = api.PcfSet(o, t, v, device=DEV)
    out = torch.empty((n, n), dtype=torch.float64, device=DEV)
    want = api.pdist(X, 1.0)
    ws = api.Workspace()
    ws.ensure(_lib.pcf_workspace_bytes(X.c_struct(), api.PCF_LP, None, 0))
    _refused(lambda: api.pdist(X, 1.0, out=out, workspace=ws))
    assert ws.planned is None
    assert torch.equal(api.pdist(X, 1.0, out=out, workspace=ws), want)
    # the planned workspace under capture: replays with eager work between
    got = torch.empty_like(out)
    g = _capture(lambda: api.pdist(X, 1.0, out=got, workspace=ws))
    for _ in range(3):
        got.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        assert torch.equal(api.pdist(X, 1.0, out=out, workspace=ws), want)


def test_other_calls_that_plan_are_refused():
    o, t, v = workloads.uniform_counts(60, 5, 40, seed=7)
    X = api.PcfSet(o, t, v, device=DEV)
    so = np.array([0, 20, 60])
    ws = api.Workspace()
    ws.ensure(1 << 22)
    G = torch.ones((60, 60), dtype=torch.float64, device=DEV)
    M = torch.empty((60, 60), dtype=torch.float64, device=DEV)
    for call in (lambda: api.gram(X, out=M, workspace=ws),
                 lambda: api.cdist(X, X, 1.0, out=M, workspace=ws),
                 lambda: api.pairwise_batched(so, X, api.PCF_LP, 1.0, workspace=ws),
                 lambda: api.pairwise_terms(X, [("lp", 1.0, None, 1.0)], out=M, workspace=ws),
                 lambda: api.pairwise_backward(X, api.PCF_GRAM, 0.0, G, workspace=ws)):
        _refused(call)
    assert torch.equal(api.pdist(X, 1.0, workspace=ws), api.pdist(X, 1.0))
