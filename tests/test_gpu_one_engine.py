"""Every ordering with one DMA engine, from prefixes and orders of the rest
(both time widths), against the C transcription of the oracle: every number of
shared positions, groups down to one task, tiles that are not full, blocks that
take several tiles, and ties (the lowest rank of equal times).  Whole numbers:
equality."""
import math

import numpy as np
import pytest

from oracle import cmodel
from oracle import model as M
from paper_1806_10113_amd import workloads as W

pytestmark = pytest.mark.gpu
MODEL = M.Model(4, 3, 3, 1)


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_10113_amd import tgo
    tgo.lib()
    return torch.device("cuda:0")


def groups(n):
    """A few ns with empty stages (many ties); milliseconds (32-bit time); equal
    tasks (every ordering ties); seconds and the longest durations (64-bit)."""
    rng = np.random.default_rng(500 + n)
    tiny = rng.integers(0, 4, size=(n, 3)).astype(np.int64)
    ms = W.single_group_mixed(n, 5)
    return [tiny, ms, np.full((n, 3), 7, dtype=np.int64), ms * 300,
            rng.integers(0, 1 << 40, size=(n, 3)).astype(np.int64)]


def check(dev, tasks):
    import torch
    from paper_1806_10113_amd import tgo
    n = len(tasks)
    ref = cmodel.exhaustive(tasks, MODEL, per_order=True)
    t = torch.as_tensor(np.ascontiguousarray(tasks)).to(dev)
    for per_order in (False, True):
        s, po = tgo.exhaustive(t, tgo.Model(2, 3, 3, 1), per_order=per_order)
        d = tgo.read_summary(s)
        assert d["status"] == 0 and d["count"] == math.factorial(n)
        for k in ("min_ns", "max_ns", "sum", "argmin_rank", "argmax_rank", "fingerprint"):
            assert d[k] == ref[k], (k, per_order)
        if per_order:
            assert np.array_equal(po.cpu().numpy(), ref["times"])


@pytest.mark.parametrize("shared", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 6, 7, 8])
def test_every_split(dev, monkeypatch, n, shared):
    monkeypatch.setenv("TGO_EXHAUSTIVE_M", str(shared))
    for tasks in groups(n):
        check(dev, tasks)


@pytest.mark.parametrize("blocks", [None, 1, 3])
@pytest.mark.parametrize("n", [7, 9])
def test_blocks_of_several_tiles(dev, monkeypatch, n, blocks):
    if blocks:
        monkeypatch.setenv("TGO_EXHAUSTIVE_BLOCKS", str(blocks))
    for tasks in groups(n):
        check(dev, tasks)
