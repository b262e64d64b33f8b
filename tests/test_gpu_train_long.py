"""Weight gradients of the largest batch with 48 chunks of rows and the smallest with
64, against 64-bit sums of the activations and activation gradients that the same
pass stored (bf16, so their products and sums are exact enough in float64)."""
import numpy as np
import pytest

from paper_1806_10113_amd import workloads as W

pytestmark = pytest.mark.gpu
OFF_W1, OFF_B1, OFF_W2, OFF_B2 = 0, 12288, 12544, 78080


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_10113_amd import tgo
    tgo.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("rows", [1 << 18, (1 << 18) + 64])
def test_long_batches(dev, rows):
    import torch
    from paper_1806_10113_amd import tgo
    b = W.batch_groups(256, 8, 16, 17, per_task_label=True)
    rng = np.random.default_rng(18)
    gid = rng.integers(0, b.n_groups, rows).astype(np.int32)
    key = rng.random((rows, 16))
    past = np.arange(16)[None, :] >= np.asarray(b.sizes())[gid][:, None]
    key[past] = 2.0
    orders = np.argsort(key, axis=1).astype(np.uint8)
    orders[past] = 255
    T = rng.integers(50_000_000, 150_000_000, rows).astype(np.int64)
    net = tgo.Surrogate(max_rows=rows, max_groups=b.n_groups)
    net.init(19)
    put = lambda a: torch.as_tensor(a).to(dev)
    grad = net.grad(put(b.tasks), put(b.offs), put(orders), put(gid), put(T))[0].double().cpu().numpy()
    val = lambda what: net.batch_values(what, rows)
    G2, G1 = val(net.BATCH_G2), val(net.BATCH_G1)
    want = {OFF_W1: G1.T @ val(net.BATCH_FEATURES), OFF_B1: G1.sum(0),
            OFF_W2: G2.T @ val(net.BATCH_H1), OFF_B2: G2.sum(0)}
    net.close()
    # a chunk adds rows / 48 / 32 float32 partial sums in turn; roundings of half an
    # ulp (2^-24 of the sum so far) that fall either way grow with the root of their number
    tol = (rows / 48 / 32) ** 0.5 * 2.0 ** -24
    for off, w in want.items():
        err = grad[off:off + w.size].reshape(w.shape) - w
        assert np.sqrt((err ** 2).mean()) <= tol * np.sqrt((w ** 2).mean()), off
