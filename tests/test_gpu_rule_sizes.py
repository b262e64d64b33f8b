"""The device-memory limit and concurrent kernels on groups of 5 to 7 tasks, where the
rule's tables before the queue have the sizes that are no multiple of a slot: every
depth, both time widths, both launch schemes, every ordering against the C
transcription of the oracle.  Whole numbers: equality."""
import math

import numpy as np
import pytest

from oracle import cmodel
from oracle import model as M
from paper_1806_10113_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_10113_amd import tgo
    tgo.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("n", [5, 6, 7])
@pytest.mark.parametrize("scale", [1, 300])  # milliseconds; seconds (64-bit time)
@pytest.mark.parametrize("engines", [2, 1])
def test_every_ordering(dev, monkeypatch, n, scale, engines):
    import torch
    from paper_1806_10113_amd import tgo
    model, m = M.Model(8, 5, 7, engines), tgo.Model(3, 5, 7, engines)
    tasks = W.single_group_mixed(n, 60 + n) * scale
    mem = W.footprints(tasks)
    cap = W.capacity_fraction(mem, 0.45)
    units = np.random.default_rng(n).integers(1, 8, n).astype(np.int32)
    t, md, ud = (torch.as_tensor(a).to(dev) for a in (tasks, mem, units))
    want = (np.asarray(cmodel.mem_times(tasks, mem, cap, model)), np.asarray(cmodel.cke_times(tasks, units, 9, model)))
    for depth in (None, 1, 2, 3, 4, 5):
        if depth:
            monkeypatch.setenv("TGO_MEM_M", str(depth))
            monkeypatch.setenv("TGO_CKE_M", str(depth))
        for times, (s, po) in zip(want, (tgo.exhaustive_mem(t, md, cap, m, per_order=True),
                                         tgo.exhaustive_cke(t, ud, 9, m, per_order=True))):
            assert np.array_equal(po.cpu().numpy(), times), depth
            d = tgo.read_summary(s)
            assert d["status"] == 0 and d["count"] == math.factorial(n)
            assert (d["min_ns"], d["argmin_rank"]) == (times.min(), times.argmin())
            assert (d["max_ns"], d["argmax_rank"]) == (times.max(), times.argmax())
