"""Whole orderings in the potential form (two DMA engines, small potentials)
and on both sides of its limit: the 32-bit limit q * bound < 2^31, the 32-bit
chain form above it, the 64-bit limit 2^51 and the chain form above that, for
rates from 1/q to 1 -- against the oracle.  Whole numbers: equality."""
import numpy as np
import pytest

from oracle import model as M

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_10113_amd import tgo
    tgo.lib()
    return torch.device("cuda:0")


RATES = [(0, 1, 1), (2, 3, 3), (3, 3, 8), (3, 8, 3), (4, 1, 16), (10, 850, 1016), (10, 1, 3)]
# largest duration: a few ns with empty stages (events at one instant), ms,
# around the 32-bit potential limit, seconds, and past 2^51 potentials
SCALES = [3, 20_000_000, 130_000_000, 60_000_000_000, (1 << 40) - 1]


@pytest.mark.parametrize("rates", RATES)
@pytest.mark.parametrize("n", [1, 2, 5, 11, 16])
def test_evaluate(dev, rates, n):
    import torch
    from paper_1806_10113_amd import tgo
    rng = np.random.default_rng(1000 * n + rates[0])
    m = M.Model(1 << rates[0], rates[1], rates[2])
    orders = np.array([rng.permutation(n) for _ in range(70)], dtype=np.uint8)
    for hi in SCALES:
        tasks = rng.integers(0, hi + 1, size=(n, 3)).astype(np.int64)
        tasks[rng.random((n, 3)) < 0.1] = 0
        got = tgo.evaluate(torch.as_tensor(tasks).to(dev), torch.as_tensor(orders).to(dev),
                           tgo.Model(*rates)).cpu().tolist()
        assert got == [M.simulate(tasks, o, m) for o in orders], hi


def test_search_takes_each_group_on_its_own_form(dev):
    """Groups of every scale in one call: the best sampled time is the one
    tgo_evaluate gives the same sample (sampled orderings read back as training
    pairs), so both agree with the oracle there."""
    import torch
    from paper_1806_10113_amd import tgo
    rng = np.random.default_rng(77)
    sizes = [16, 9, 16, 4, 12]
    groups = [rng.integers(0, hi + 1, size=(n, 3)).astype(np.int64) for n, hi in zip(sizes, SCALES)]
    tasks = torch.as_tensor(np.concatenate(groups)).to(dev)
    offs = torch.as_tensor(np.cumsum([0] + sizes).astype(np.int32)).to(dev)
    per = 192
    orders, gid, T, status = tgo.pairs(tasks, offs, per, seed=5)
    assert status.cpu().tolist() == [0] * len(sizes)
    res = tgo.read_search(tgo.random_search(tasks, offs, per, seed=5))
    o, t = orders.cpu().numpy(), T.cpu().numpy()
    for g, n in enumerate(sizes):
        rows = slice(g * per, (g + 1) * per)
        want = [M.simulate(groups[g], x[:n], M.DEFAULT) for x in o[rows]]
        assert t[rows].tolist() == want
        assert res[g]["cand_best_ns"] == min(want) and res[g]["best_sample"] == int(np.argmin(want))
