"""Evaluation of many orderings of small groups: rows of every length that is read by
4, 8 or 16 loads, on both sides of the group size up to which one launch serves
both time widths and of the row count where larger groups get two, with rows that
are no permutations among them, against the oracle."""
import itertools

import numpy as np
import pytest

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


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 8, 9])
@pytest.mark.parametrize("scale", [1, 200])  # milliseconds; seconds (64-bit time)
@pytest.mark.parametrize("engines", [2, 1])
def test_many_short_rows(dev, n, scale, engines):
    import torch
    from paper_1806_10113_amd import tgo
    tasks = W.single_group_mixed(n, 30 + n) * scale
    model = M.Model(8, 5, 6, engines)
    perms = np.array(list(itertools.islice(itertools.permutations(range(n)), 120)), dtype=np.uint8)
    bad = []
    for j in range(n):  # a value past the group, past a nibble, and twice
        for v in (n, 16 + j, 255) + ((int(perms[0, j - 1]),) if n > 1 else ()):
            bad.append(perms[0].copy())
            bad[-1][j] = v
    rows = np.concatenate([perms, np.array(bad, dtype=np.uint8)])
    want = np.array([M.simulate(tasks, o, model) for o in perms] + [tgo.TGO_EINVAL] * len(bad))
    t, o = torch.as_tensor(tasks).to(dev), torch.as_tensor(rows).to(dev)
    for m in (len(rows), 131071, 131073, 1000003):
        got = tgo.evaluate(t, o.repeat(m // len(rows) + 1, 1)[:m].contiguous(), tgo.Model(3, 5, 6, engines))
        assert np.array_equal(got.cpu().numpy(), np.resize(want, m)), m
