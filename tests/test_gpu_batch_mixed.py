"""Batches that put groups of 12 tasks (chain form, the longest queue) beside groups
of 1 to 11 (potential form up to 10 where the rates allow it) on the waves of one
block, in several orders: every group as in a batch of its own, the groups of 12 as
the single-group search finds them, the others as the C transcription of the oracle
does.  Whole numbers: equality."""
import numpy as np
import pytest

from oracle import cmodel
from oracle import model as M
from paper_1806_10113_amd import workloads as W

pytestmark = pytest.mark.gpu
FIELDS = ("status", "count", "min_ns", "max_ns", "sum", "argmin_rank", "argmax_rank", "fingerprint", "best", "worst")


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_10113_amd import tgo
    tgo.lib()
    return torch.device("cuda:0")


def run(dev, model, gs, desc=None):
    import torch
    from paper_1806_10113_amd import tgo
    offs = np.cumsum([0] + [len(g) for g in gs]).astype(np.int32)
    plan = tgo.Plan(model, max_groups=len(gs))
    if desc:
        plan.set_decomposition({**plan.describe(), **desc})
    out = plan.run(torch.as_tensor(np.concatenate(gs)).to(dev), torch.as_tensor(offs).to(dev))
    res = [tgo.read_summary(row) for row in out]
    plan.close()
    return [{k: d[k] for k in FIELDS} for d in res]


# rates with slack in the overlapped DtHs (p_dth > 1); the last one is 1/1024ths,
# where only the smallest groups take the potential form
@pytest.mark.parametrize("rates", [(2, 3, 3), (3, 5, 7), (10, 850, 200)])
@pytest.mark.parametrize("seed", [0, 1])
def test_largest_groups_beside_smaller_ones(dev, rates, seed):
    import torch
    from paper_1806_10113_amd import tgo
    rng = np.random.default_rng(900 + seed)
    model, ref = tgo.Model(*rates), M.Model(1 << rates[0], rates[1], rates[2])
    scale = 1 if rates[0] < 10 else 40  # 1/1024ths: the form ends at 2 ms a group
    gs = [W.single_group_mixed(12, 10 * seed + i) // scale for i in range(4)]
    gs += [W.single_group_mixed(n, 100 * seed + i) // scale for i, n in enumerate(rng.integers(1, 11, 60))]
    gs += [W.single_group_mixed(n, 100 * seed + 70 + i) // scale for i, n in enumerate((8, 9, 9, 10, 10, 10, 11))]
    want = []
    for g in gs:
        alone = run(dev, model, [g])[0]
        if len(g) < 11:
            d = cmodel.exhaustive(g, ref)
        else:
            d = tgo.read_summary(tgo.exhaustive(torch.as_tensor(g).to(dev), model)[0])
        for k in ("min_ns", "max_ns", "sum", "argmin_rank", "argmax_rank", "fingerprint"):
            assert alone[k] == d[k], (k, len(g))
        want.append(alone)
    perms = [np.arange(len(gs)), np.argsort([-len(g) for g in gs], kind="stable")]
    perms += [rng.permutation(len(gs)) for _ in range(3)]
    for perm in perms:
        for desc in (None, {"lane_mult": 1}, {"lane_mult": 4, "blocks": 512}):
            got = run(dev, model, [gs[i] for i in perm], desc)
            for i, d in zip(perm, got):
                assert d == want[i], (len(gs[i]), desc)
