"""Plans that travel as kernel arguments (one, two and three launches) and by
copy: batches whose plan sizes lie on either side of each limit, and sets whose
rows are packed by 16 and by 64 lanes a PCF, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_07183_amd import api, workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("problems", [1, 36, 41, 83, 88, 126, 133])
@pytest.mark.parametrize("lo,hi", [(1, 20), (30, 60)])
def test_batch_plan_sizes(problems, lo, hi):
    o, t, v = workloads.uniform_counts(5 * problems, lo, hi, seed=problems)
    X = api.PcfSet(o, t, v, device=DEV)
    so = 5 * np.arange(problems + 1)
    out, oo = api.pairwise_batched(so, X, api.PCF_LP, 1.0)
    out = out.cpu().numpy()
    i, j = np.meshgrid(np.arange(5), np.arange(5), indexing="ij")
    I = (so[:-1, None] + i.ravel()[None, :]).ravel()
    J = (so[:-1, None] + j.ravel()[None, :]).ravel()
    ref, ab = oracle.entries(oracle.LP, 1.0, o, t, v, I, J, with_abs=True)
    assert np.all(np.abs(out - ref) <= 1e-12 * np.maximum(ab, 1e-300))


def test_overlapped_calls_keep_their_plans():
    # calls enqueued without waiting: each plan is the one its call was given
    sets = []
    for seed, n in enumerate([7, 40, 130, 65]):
        o, t, v = workloads.uniform_counts(n, 2, 90, seed=200 + seed)
        sets.append((o, t, v, api.PcfSet(o, t, v, device=DEV)))
    ws = api.Workspace()
    ws.ensure(1 << 22)
    outs = [api.pdist(X, 1.0, workspace=ws) for _ in range(3) for _, _, _, X in sets]
    torch.cuda.synchronize()
    for k, M in enumerate(outs):
        o, t, v, _ = sets[k % len(sets)]
        R = oracle.matrix(oracle.LP, 1.0, o, t, v)
        assert np.all(np.abs(M.cpu().numpy() - R) <= 1e-12 * np.maximum(R, 1e-300))
