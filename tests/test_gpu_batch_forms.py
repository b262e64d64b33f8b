"""Batches whose groups take different forms of the walk in one launch (the
potential form up to 10 tasks where rates and sizes fit, else the chain form, or
64-bit time), for every depth, against the C transcription of the oracle.  Whole
numbers: equality."""
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


def groups(rates):
    """Sizes 1 to 9: a few ns with empty stages; milliseconds; the time bound just
    below and just above 2^31 / q (the limit of the potential form); seconds."""
    rng = np.random.default_rng(31 + rates[1])
    q = 1 << rates[0]
    out = []
    for n in (1, 2, 3, 5, 7, 8, 9):
        edge = int((1 << 31) / q / n / (q / rates[1] + 1 + q / rates[2])) + 2
        tiny = rng.integers(0, 4, size=(n, 3)).astype(np.int64)
        out += [tiny, W.single_group_mixed(n, n), rng.integers(edge * 9 // 10, edge * 49 // 50, size=(n, 3)),
                rng.integers(edge * 51 // 50, edge * 11 // 10 + 1, size=(n, 3)), W.single_group_mixed(n, n) * 300]
    order = rng.permutation(len(out))
    return [np.asarray(out[i], dtype=np.int64) for i in order]


@pytest.mark.parametrize("rates", [(2, 3, 3), (4, 9, 13), (3, 2, 1), (10, 850, 870), (0, 1, 1)])
@pytest.mark.parametrize("depth", [None, 1, 2, 3, 4, 5])
def test_forms_side_by_side(dev, rates, depth):
    import torch
    from paper_1806_10113_amd import tgo
    gs = groups(rates)
    if depth in (1, 2):  # few positions walked: many subtrees
        gs = [g for g in gs if len(g) <= 8]
    if depth is None and rates == (2, 3, 3):  # the largest group of the potential form and the next
        gs += [W.single_group_mixed(10, 5), W.single_group_mixed(11, 5)]
    offs = np.cumsum([0] + [len(g) for g in gs]).astype(np.int32)
    plan = tgo.Plan(tgo.Model(*rates), max_groups=len(gs))
    if depth:
        desc = plan.describe()
        desc.update(m_by_n=[min(n, depth) for n in range(1, 13)], lane_mult=2)
        plan.set_decomposition(desc)
    out = plan.run(torch.as_tensor(np.concatenate(gs)).to(dev), torch.as_tensor(offs).to(dev))
    model = M.Model(1 << rates[0], rates[1], rates[2])
    for g, row in zip(gs, out):
        d = tgo.read_summary(row)
        ref = cmodel.exhaustive(g, model)
        assert d["status"] == 0 and d["count"] == math.factorial(len(g))
        for k in ("min_ns", "max_ns", "sum", "argmin_rank", "argmax_rank", "fingerprint"):
            assert d[k] == ref[k], (k, len(g), g.max())
    plan.close()
