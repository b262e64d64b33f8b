"""tgo_evaluate reads each row once, as bytes at any address: alignment, row
counts and invalid values against the oracle (whole numbers: equality)."""
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


@pytest.mark.parametrize("n", [1, 2, 7, 15, 16])
def test_evaluate_rows_at_any_alignment(dev, n):
    """Rows that start at an odd address, fewer rows than a block and more
    than the resident blocks take at once, invalid values in every byte."""
    import torch
    from paper_1806_10113_amd import tgo
    rng = np.random.default_rng(900 + n)
    tasks = W.batch_groups(1, n, n, 900 + n, per_task_label=True).tasks
    t = torch.as_tensor(tasks).to(dev)
    rows = np.array([rng.permutation(n) for _ in range(301)], dtype=np.uint8)
    bad = rows[:n].copy()
    for j in range(n):  # a repeated task, a value past n, one past 15
        bad[j, j] = (bad[j, j] + 1) % n if n > 1 else 1
    big = rows[:n].copy()
    big[np.arange(n), np.arange(n)] = [16 + 17 * j % 240 for j in range(n)]
    orders = np.concatenate([rows, bad, big])
    want = [M.simulate(tasks, o, M.DEFAULT) for o in rows] + [tgo.TGO_EINVAL] * (2 * n)
    flat = torch.zeros(orders.size + 3, dtype=torch.uint8, device=dev)
    for off in range(4):
        flat[off:off + orders.size] = torch.as_tensor(orders.reshape(-1)).to(dev)
        o = flat[off:off + orders.size].reshape(orders.shape)
        assert tgo.evaluate(t, o).cpu().tolist() == want, off
    reps = 4000  # 1.2 million rows: every lane takes several
    got = tgo.evaluate(t, torch.as_tensor(rows).to(dev).repeat(reps, 1)).cpu().numpy()
    assert np.array_equal(got, np.tile(np.array(want[:len(rows)]), reps))


@pytest.mark.parametrize("rows", [1, 256, 257, 131072, 131073])
@pytest.mark.parametrize("scale", [1, 300, -1])
def test_one_launch_or_two(dev, rows, scale):
    """Row counts around a block and around the last that both time widths share
    a launch for: 32-bit time, 64-bit time (tasks of seconds) and a group in error."""
    import torch
    from paper_1806_10113_amd import tgo
    rng = np.random.default_rng(rows)
    tasks = W.batch_groups(1, 9, 9, 7, per_task_label=True).tasks * scale
    few = np.array([rng.permutation(9) for _ in range(min(rows, 97))], dtype=np.uint8)
    orders = np.resize(few, (rows, 9))
    got = tgo.evaluate(torch.as_tensor(tasks).to(dev), torch.as_tensor(orders).to(dev)).cpu().numpy()
    want = [M.simulate(tasks, o, M.DEFAULT) if scale > 0 else tgo.TGO_ERANGE for o in few]
    assert np.array_equal(got, np.resize(np.array(want), rows))
