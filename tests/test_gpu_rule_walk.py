"""The enumerations under a start rule (device memory, concurrent kernels):
every depth of the walk, both time widths, with and without the per-ordering
output, against the C transcription of the oracle.  Whole numbers: equality."""
import math

import numpy as np
import pytest

from oracle import cmodel
from oracle import model as M
from paper_1806_10113_amd import workloads as W

pytestmark = pytest.mark.gpu
N = 8  # 40,320 orderings: also the largest group of the one-lane-per-ordering kernel
MODELS = [M.DEFAULT, M.Model(16, 9, 13), M.NO_SLOWDOWN, M.Model(4, 3, 3, 1)]


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_10113_amd import tgo
    tgo.lib()
    return torch.device("cuda:0")


def to_dev(a, dev):
    import torch
    return torch.as_tensor(np.ascontiguousarray(a)).to(dev)


def groups():
    """(tasks, footprints, memory capacity, units, unit capacity): milliseconds
    (32-bit time), a few ns with empty stages (events at the same instant),
    seconds (64-bit time)."""
    rng = np.random.default_rng(81)
    ms = W.single_group_mixed(N, 5)
    tiny = rng.integers(0, 4, size=(N, 3)).astype(np.int64)
    out = []
    for tasks, frac in ((ms, 0.35), (tiny, 0.5), (ms * 300, 0.6)):
        mem = W.footprints(tasks) + rng.integers(0, 3, N)
        out.append((tasks, mem, W.capacity_fraction(mem, frac), rng.integers(1, 8, N).astype(np.int32), 9))
    return out


def check(summary, po, times):
    from paper_1806_10113_amd import tgo
    assert np.array_equal(po.cpu().numpy(), times)
    for s in summary:
        d = tgo.read_summary(s)
        assert d["status"] == 0 and d["count"] == math.factorial(N)
        assert (d["min_ns"], d["argmin_rank"]) == (times.min(), times.argmin())
        assert (d["max_ns"], d["argmax_rank"]) == (times.max(), times.argmax())
        assert d["sum"] == int(times.sum())
        assert d["fingerprint"] == sum((2 * r + 1) * int(x) for r, x in enumerate(times)) % (1 << 64)


@pytest.mark.parametrize("depth", [None, 1, 2, 3, 4, 5])
@pytest.mark.parametrize("model", MODELS)
def test_every_depth(dev, monkeypatch, depth, model):
    from paper_1806_10113_amd import tgo
    if depth:
        monkeypatch.setenv("TGO_MEM_M", str(depth))
        monkeypatch.setenv("TGO_CKE_M", str(depth))
    m = tgo.Model(int(math.log2(model.q)), model.p_htd, model.p_dth, model.dma_engines)
    for tasks, mem, mcap, units, ucap in groups():
        t, md, ud = to_dev(tasks, dev), to_dev(mem, dev), to_dev(units, dev)
        s, po = tgo.exhaustive_mem(t, md, mcap, m, per_order=True)
        s2, _ = tgo.exhaustive_mem(t, md, mcap, m)
        check((s, s2), po, np.asarray(cmodel.mem_times(tasks, mem, mcap, model)))
        s, po = tgo.exhaustive_cke(t, ud, ucap, m, per_order=True)
        s2, _ = tgo.exhaustive_cke(t, ud, ucap, m)
        check((s, s2), po, np.asarray(cmodel.cke_times(tasks, units, ucap, model)))


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("model", MODELS)
def test_small_groups_take_either_path(dev, monkeypatch, n, model):
    """One lane per ordering (one block up to n = 6, several above) against
    the general walk: every field of the summary and every time."""
    from paper_1806_10113_amd import tgo
    m = tgo.Model(int(math.log2(model.q)), model.p_htd, model.p_dth, model.dma_engines)
    for tasks, mem, mcap, units, ucap in groups():
        t, md, ud = to_dev(tasks[:n], dev), to_dev(mem[:n], dev), to_dev(units[:n], dev)

        def runs():
            out = []
            for s, po in (tgo.exhaustive(t, m, per_order=True), tgo.exhaustive(t, m),
                          tgo.exhaustive_mem(t, md, mcap, m, per_order=True),
                          tgo.exhaustive_cke(t, ud, ucap, m, per_order=True)):
                out.append((tgo.read_summary(s), None if po is None else po.cpu().tolist()))
            return out

        small = runs()
        for k in ("TGO_EXHAUSTIVE_M", "TGO_MEM_M", "TGO_CKE_M"):
            monkeypatch.setenv(k, "1")
        assert small == runs()
        for k in ("TGO_EXHAUSTIVE_M", "TGO_MEM_M", "TGO_CKE_M"):
            monkeypatch.delenv(k)


def test_depths_agree_on_a_large_group(dev, monkeypatch):
    """n = 11 (waves of lanes that share a prefix set): every depth gives the
    summary of depth 1."""
    from paper_1806_10113_amd import tgo
    tasks = W.single_group_mixed(11, 9)
    mem = W.footprints(tasks)
    units = np.random.default_rng(82).integers(1, 8, 11).astype(np.int32)
    t, md, ud = to_dev(tasks, dev), to_dev(mem, dev), to_dev(units, dev)
    for engines in (2, 1):
        m = tgo.Model(2, 3, 3, engines)
        want = None
        for depth in (1, 2, 3, 4, 5):
            monkeypatch.setenv("TGO_MEM_M", str(depth))
            monkeypatch.setenv("TGO_CKE_M", str(depth))
            got = (tgo.read_summary(tgo.exhaustive_mem(t, md, W.capacity_fraction(mem, 0.4), m)[0]),
                   tgo.read_summary(tgo.exhaustive_cke(t, ud, 10, m)[0]))
            want = want or got
            assert got == want, (engines, depth)
