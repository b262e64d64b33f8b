"""NoReorder and the Heuristic setup on the window formulation: every depth of
the last round's walk and both time widths against the oracle (whole numbers:
equality), with empty stages so that several commands meet at one instant."""
import math

import numpy as np
import pytest

from oracle import model as M
from oracle import rounds as OR
from paper_1806_10113_amd import workloads as W

pytestmark = pytest.mark.gpu
MODELS = [M.DEFAULT, M.Model(16, 9, 13), M.Model(4, 3, 3, 1)]


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_10113_amd import tgo
    tgo.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("T,R", [(3, 2), (4, 2), (2, 4), (4, 1)])
@pytest.mark.parametrize("depth", [None, 1, 2, 3, 4])
def test_every_depth(dev, monkeypatch, T, R, depth):
    import torch
    from paper_1806_10113_amd import tgo
    if depth and depth > T:
        pytest.skip("no deeper than a round")
    if depth:
        monkeypatch.setenv("TGO_ROUNDS_M", str(depth))
    rng = np.random.default_rng(100 * T + R)
    paper = W.rounds_experiment("BK50", T, R, 7)
    for tasks in (paper, rng.integers(0, 4, size=(T * R, 3)).astype(np.int64), paper * 200):
        t = torch.as_tensor(np.ascontiguousarray(tasks)).to(dev)
        for model in MODELS:
            m = tgo.Model(int(math.log2(model.q)), model.p_htd, model.p_dth, model.dma_engines)
            s, po, g = tgo.rounds(t, T, R, m, per_order=True)
            s2, _, _ = tgo.rounds(t, T, R, m)
            ref = OR.noreorder_summary([tuple(x) for x in tasks.tolist()], T, R, model)
            heur = OR.heuristic_setup(tasks.tolist(), T, R, model)
            assert np.array_equal(po.cpu().numpy(), np.asarray(ref["times"])), (model, tasks.max())
            for d in (tgo.read_summary(s), tgo.read_summary(s2)):
                for k in ("min_ns", "argmin_rank", "max_ns", "argmax_rank", "fingerprint", "sum", "count"):
                    assert int(d[k]) == int(ref[k]), k
                assert d["heur_ns"] == heur[0]
                assert d["heur"] == [x for _, o in heur[1] for x in o]
