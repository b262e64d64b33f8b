"""The training kernels at the edges of their tiles, every stage against the
float64 oracle: half a row block (64 rows), an odd number of halves, one K chunk
and the first row of the next, and more rows than the smallest chunks cover
(48 x 256 and 64 more)."""
import numpy as np
import pytest

import test_gpu_surrogate as base

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_10113_amd import tgo
    tgo.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("groups", [1, 3, 4, 5, 193])
def test_every_stage(dev, monkeypatch, groups):
    from paper_1806_10113_amd import tgo
    whole = tgo.Surrogate
    monkeypatch.setattr(tgo, "Surrogate", lambda max_rows, max_groups: whole(max_rows=12352, max_groups=max_groups))
    base.test_gradients_stage_by_stage(dev, groups, 64)


def test_first_rows_of_a_batch(dev):
    """Reading back the first rows gives the first rows of reading all."""
    sur, *_ = base._grad_case(dev, 3, 64, 302, 13, 2)
    for what in (sur.BATCH_FEATURES, sur.BATCH_H1, sur.BATCH_G1):
        whole = sur.batch_values(what, 192)
        for rows in (1, 17, 64, 65, 190):
            assert np.array_equal(sur.batch_values(what, rows), whole[:rows])
    sur.close()
