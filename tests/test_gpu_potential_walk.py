"""The walk of two-engine groups in the potential form (depth 5) against the C
transcription of the oracle: every rate that takes it and those that do not
(p_htd = q, slack sums of 256 and more), the largest potentials that fit and the
first that do not, empty stages, the smallest groups of that depth and the first
that take it by themselves.  Whole numbers: equality."""
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


# (log2 q, p_htd, p_dth); q - p_htd odd, even, a power of two, 1 and 0
RATES = [(2, 3, 3), (10, 850, 870), (10, 850, 21), (4, 9, 13), (2, 3, 4), (3, 2, 1), (10, 1, 1), (10, 1023, 37), (6, 64, 50), (0, 1, 1)]


def tasks_of(n, rates, rng):
    """A few ns with empty stages; milliseconds; the group's time bound (every
    transfer at its overlapped rate) just below and just above 2^31 / q, the
    limit of q times it."""
    tiny = rng.integers(0, 4, size=(n, 3)).astype(np.int64)
    ms = W.single_group_mixed(n, 5)
    q = 1 << rates[0]
    edge = int((1 << 31) / q / n / (q / rates[1] + 1 + q / rates[2]))
    below = rng.integers(edge * 9 // 10, edge * 49 // 50, size=(n, 3)).astype(np.int64)
    above = rng.integers(edge * 51 // 50, edge * 11 // 10, size=(n, 3)).astype(np.int64)
    mixed = below.copy()
    mixed[rng.random((n, 3)) < 0.3] = 0
    return [tiny, ms, below, above, mixed]


def check(dev, tasks, m, model, per_order=True):
    import torch
    from paper_1806_10113_amd import tgo
    n = len(tasks)
    t = torch.as_tensor(np.ascontiguousarray(tasks)).to(dev)
    s, _ = tgo.exhaustive(t, m)
    d = tgo.read_summary(s)
    ref = cmodel.exhaustive(tasks, model, per_order=per_order)
    assert d["status"] == 0 and d["count"] == math.factorial(n)
    for k in ("min_ns", "max_ns", "sum", "argmin_rank", "argmax_rank", "fingerprint"):
        assert d[k] == ref[k], k
    if per_order:
        s, po = tgo.exhaustive(t, m, per_order=True)
        assert np.array_equal(po.cpu().numpy(), ref["times"])
        assert tgo.read_summary(s) == d


@pytest.mark.parametrize("n", [5, 6, 8])
@pytest.mark.parametrize("rates", RATES)
def test_depth_five(dev, monkeypatch, n, rates):
    from paper_1806_10113_amd import tgo
    monkeypatch.setenv("TGO_EXHAUSTIVE_M", "5")
    rng = np.random.default_rng(100 * n + rates[1])
    model = M.Model(1 << rates[0], rates[1], rates[2])
    for tasks in tasks_of(n, rates, rng):
        check(dev, tasks, tgo.Model(*rates), model)


def test_first_group_that_takes_it(dev):
    from paper_1806_10113_amd import tgo
    rng = np.random.default_rng(11)
    for tasks in tasks_of(11, (2, 3, 3), rng)[1:3]:
        check(dev, tasks, tgo.Model(), M.DEFAULT, per_order=False)


@pytest.mark.parametrize("swap", [False, True])
def test_twelve_tasks_either_way(dev, monkeypatch, swap):
    """From 12 tasks on the form depends on the DtHs' share of the transfers: the
    same group with HtDs and DtHs exchanged takes one form and then the other."""
    import torch
    from paper_1806_10113_amd import tgo
    tasks = W.single_group_mixed(12, 5)
    tasks[:, 0] *= 2
    if swap:
        tasks = np.ascontiguousarray(tasks[:, ::-1])
    s, _ = tgo.exhaustive(torch.as_tensor(tasks).to(dev), tgo.Model())
    d = tgo.read_summary(s)
    model = M.DEFAULT
    assert d["status"] == 0 and d["count"] == math.factorial(12)
    # a sample of ranks bounds the extremes, and the reported orderings attain them
    lo = cmodel.exhaustive(tasks, model, stride=7919)
    assert d["min_ns"] <= lo["min_ns"] and d["max_ns"] >= lo["max_ns"]
    for key, rank in (("min_ns", "argmin_rank"), ("max_ns", "argmax_rank")):
        one = cmodel.exhaustive(tasks, model, lo=int(d[rank]), hi=int(d[rank]) + 1)
        assert one["min_ns"] == d[key]
    # exchanging the walk's depth exchanges the kernel, not the answer
    monkeypatch.setenv("TGO_EXHAUSTIVE_M", "4")
    s4, _ = tgo.exhaustive(torch.as_tensor(tasks).to(dev), tgo.Model())
    assert tgo.read_summary(s4) == d
