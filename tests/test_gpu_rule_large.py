"""Concurrent kernels and the memory limit on a group of 11 tasks, where the deepest
walk runs (its state spills): the summary over all 39,916,800 orderings against the
C transcription of the oracle, two engines, several rates.  Whole numbers: equality."""
import math

import numpy as np
import pytest

from oracle import cmodel
from oracle import model as M
from paper_1806_10113_amd import workloads as W

pytestmark = pytest.mark.gpu
N = 11


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_10113_amd import tgo
    tgo.lib()
    return torch.device("cuda:0")


def check(d, times):
    assert d["status"] == 0 and d["count"] == len(times) == math.factorial(N)
    lo, hi = int(times.argmin()), int(times.argmax())
    assert (d["min_ns"], d["argmin_rank"]) == (int(times[lo]), lo)
    assert (d["max_ns"], d["argmax_rank"]) == (int(times[hi]), hi)
    assert d["sum"] == int(times.sum())
    r = np.arange(len(times), dtype=np.uint64)
    assert d["fingerprint"] == int(((2 * r + 1) * times.astype(np.uint64)).sum(dtype=np.uint64))


@pytest.mark.parametrize("rates", [(2, 3, 3), (3, 5, 7)])
@pytest.mark.parametrize("rule", ["memory", "concurrent"])
def test_every_ordering(dev, rates, rule):
    import torch
    from paper_1806_10113_amd import tgo
    model, m = M.Model(1 << rates[0], rates[1], rates[2]), tgo.Model(*rates)
    tasks = W.single_group_mixed(12, seed=4)[:N]
    t = torch.as_tensor(tasks).to(dev)
    if rule == "memory":
        mem = W.footprints(tasks)
        cap = W.capacity_fraction(mem, 0.4)
        s, _ = tgo.exhaustive_mem(t, torch.as_tensor(mem).to(dev), cap, m)
        want = cmodel.mem_times(tasks, mem, cap, model)
    else:
        units = np.random.default_rng(5).integers(1, 8, N).astype(np.int32)
        s, _ = tgo.exhaustive_cke(t, torch.as_tensor(units).to(dev), 10, m)
        want = cmodel.cke_times(tasks, units, 10, model)
    check(tgo.read_summary(s), np.asarray(want))
