"""Performance cases of the task-group library: what its users call, over the
sizes they call it with.

A case names an operation ("op") and its sizes.  `prepare` makes the inputs
from the seed and whatever a program keeps between calls (device tensors, a
batch plan, network weights); `run` is one pass through the public entry
points.  Every operation but "grad" returns whole numbers only (total times in
ns, orderings, packed result records), which have one right value.

Tasks come from the repository's seeded generators: dominant-kernel and
dominant-transfer tasks of 0.1-20 ms per command, the BK benchmarks for groups
of four and for dependent tasks.  `long` tasks are 100 times longer, which
takes a group past the 32-bit time range.
"""
import math

import numpy as np
import torch

from paper_1806_10113_amd import tgo, workloads as W

PARAMS = ((256, 48), (256,), (256, 256), (256,), (256, 256), (256,), (256,), (1,))


def listed():
    return [
        # the paper's own groups: four tasks, every ordering and Algorithm 1;
        # the smallest call, where launches and latency count
        {"name": "group-n4", "op": "group", "n": 4, "engines": 2},
        # the headline: every ordering of 12 mixed tasks and Algorithm 1
        {"name": "group-n12", "op": "group", "n": 12, "engines": 2},
        # the largest group that is enumerated, devices with one DMA engine
        {"name": "group-n13-one-dma", "op": "group", "n": 13, "engines": 1},
        # the total time of every ordering written out (distributions over the
        # orderings, as in the paper's figures), tasks of seconds: 64-bit time
        {"name": "per-order-n10-long", "op": "per_order", "n": 10, "engines": 2, "long": True},
        # a proxy's backlog: thousands of uneven groups in one call of a tuned plan
        {"name": "batch-4096", "op": "batch", "groups": 4096, "n_lo": 4, "n_hi": 10, "engines": 2},
        # given orderings of the largest group, an odd count
        {"name": "evaluate-n16", "op": "evaluate", "n": 16, "rows": 1000003, "engines": 2, "long": False},
        # a device-memory limit of 40 % of the group's footprint
        {"name": "memory-n12", "op": "memory", "n": 12, "engines": 2, "percent": 40},
        # concurrent kernels, each holding a part of the device's 256 compute units
        {"name": "concurrent-n12", "op": "concurrent", "n": 12, "engines": 2, "capacity": 256},
        # four workers with four dependent tasks each, the paper's largest shape
        {"name": "rounds-4x4", "op": "rounds", "workers": 4, "rounds": 4, "engines": 2},
        # groups too large to enumerate: sampled orderings scored exactly
        {"name": "random-search-1024", "op": "random_search", "groups": 1024, "n_lo": 16, "n_hi": 16,
         "samples": 16384},
        # the same through the learned proposal, top 64 re-scored exactly
        {"name": "proposal-1024", "op": "proposal", "groups": 1024, "n_lo": 8, "n_hi": 16, "samples": 4096},
        # one training batch of the proposal network: forward, backward, gradients
        {"name": "grad-65536", "op": "grad", "groups": 2048, "n_lo": 8, "n_hi": 16, "rows": 65536},
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(("group", "group", "per_order", "batch", "evaluate", "memory", "concurrent", "rounds",
                     "random_search", "proposal", "grad"))
    engines = rng.choice((2, 2, 1))
    c = {"op": op}
    if op not in ("random_search", "proposal", "grad"):  # overlap rates in eighths
        c.update(p_htd=rng.randint(3, 8), p_dth=rng.randint(3, 8))
    if op == "group":
        c.update(n=rng.randint(2, 12), engines=engines)
    elif op == "per_order":
        c.update(n=rng.randint(4, 10), engines=engines, long=rng.random() < 0.5)
    elif op == "batch":
        lo = rng.randint(2, 8)
        c.update(groups=_log(rng, 3, 4096), n_lo=lo, n_hi=rng.randint(lo, 10), engines=engines)
    elif op == "evaluate":
        c.update(n=rng.randint(3, 16), rows=_log(rng, 1, 2000000), engines=engines, long=rng.random() < 0.3)
    elif op == "memory":
        c.update(n=rng.randint(3, 12), engines=engines, percent=rng.choice((0, 25, 40, 60, 100)))
    elif op == "concurrent":
        c.update(n=rng.randint(3, 12), engines=engines, capacity=rng.choice((4, 32, 256)))
    elif op == "rounds":
        w, r = rng.choice(((4, 1), (4, 2), (4, 3), (4, 4), (6, 1), (6, 2), (8, 1), (3, 5), (5, 3), (2, 8)))
        c.update(workers=w, rounds=r, engines=engines)
    elif op == "grad":
        lo = rng.randint(4, 16)
        c.update(groups=_log(rng, 16, 4096), n_lo=lo, n_hi=rng.randint(lo, 16), rows=64 * _log(rng, 1, 1024))
    else:
        lo = rng.randint(4, 16)
        groups = _log(rng, 1, 1024)
        c.update(groups=groups, n_lo=lo, n_hi=rng.randint(lo, 16),
                 samples=_log(rng, 64, (16384 if op == "random_search" else 4096) * 1024 // groups))
    return c


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to("cuda")


def _group(case, seed):
    """Tasks of one group: a BK benchmark's for four, else half dominant-kernel, half dominant-transfer."""
    n = case["n"]
    if n == 4 and not case.get("long"):
        return W.rounds_experiment("BK50", 4, 1, seed)
    return W.single_group_mixed(n, seed) * (100 if case.get("long") else 1)


def _groups(case, seed):
    b = W.batch_groups(case["groups"], case["n_lo"], case["n_hi"], seed, per_task_label=True)
    return b, _dev(b.tasks), _dev(b.offs)


def _orders(rng, sizes):
    """One uniform ordering per row, row i of sizes[i] tasks, padded with 255 to 16."""
    key = rng.random((len(sizes), 16))
    key[np.arange(16)[None, :] >= sizes[:, None]] = 2.0
    o = np.argsort(key, axis=1).astype(np.uint8)
    o[np.arange(16)[None, :] >= sizes[:, None]] = 255
    return o


def _weights(seed):
    """Network parameters in the library's order, float32: uniform, small biases."""
    rng = np.random.default_rng(seed + 77)
    out = []
    for i, s in enumerate(PARAMS):
        fan = 48 if i == 0 else 256
        a = math.sqrt(6.0 / fan) if i in (0, 2, 4, 6) else 0.05
        out.append(rng.uniform(-a, a, s).astype(np.float32))
    return out


def _surrogate(case, seed, rows):
    s = tgo.Surrogate(max_rows=rows, max_groups=case["groups"])
    s.set_params(np.concatenate([w.reshape(-1) for w in _weights(seed)]))
    return s


def _lower_bound(t):
    """Largest machine lower bound of a group (int64 [n, 3])."""
    h, k, d = t[:, 0], t[:, 1], t[:, 2]
    return max(1, int(h.sum() + (k + d).min()), int(h.min() + k.sum() + d.min()), int((h + k).min() + d.sum()))


def _training_batch(case, seed):
    """Shuffled (ordering, total time) pairs: times from the group's lower bound up to 1.8 times it."""
    b = W.batch_groups(case["groups"], case["n_lo"], case["n_hi"], seed, per_task_label=True)
    rng = np.random.default_rng(seed + 5)
    gid = rng.integers(0, b.n_groups, case["rows"]).astype(np.int32)
    orders = _orders(rng, b.sizes()[gid])
    lb = np.array([_lower_bound(b.group(g)) for g in range(b.n_groups)], dtype=np.int64)
    T = np.rint(lb[gid] * rng.uniform(1.0, 1.8, case["rows"])).astype(np.int64)
    return b, gid, orders, lb, T


def prepare(case, seed):
    op = case["op"]
    s = {"op": op, "seed": seed, "case": case}
    if "engines" in case:  # overlapped transfers at 6/8 of solo speed each, unless the case says otherwise
        s["model"] = tgo.Model(3, case.get("p_htd", 6), case.get("p_dth", 6), dma_engines=case["engines"])
    rng = np.random.default_rng(seed + 5)
    if op in ("group", "per_order", "evaluate", "memory", "concurrent"):
        t = _group(case, seed)
        s["tasks"] = _dev(t)
        if op == "group":
            s["offs"] = _dev(np.array([0, case["n"]], dtype=np.int32))
        elif op == "evaluate":
            o = _orders(rng, np.full(case["rows"], case["n"]))
            s["orders"] = _dev(o[:, :case["n"]])
        elif op == "memory":
            mem = W.footprints(t)
            s["mem"], s["capacity"] = _dev(mem), W.capacity_fraction(mem, case["percent"] / 100)
        elif op == "concurrent":
            s["units"] = _dev(rng.integers(1, case["capacity"] + 1, case["n"]).astype(np.int32))
    elif op == "batch":
        _, s["tasks"], s["offs"] = _groups(case, seed)
        s["plan"] = tgo.Plan(s["model"], max_groups=case["groups"])
        s["plan"].autotune(s["tasks"], s["offs"])
    elif op == "rounds":
        bk = ("BK25", "BK50", "BK75")[seed % 3]
        s["tasks"] = _dev(W.rounds_experiment(bk, case["workers"], case["rounds"], seed))
    elif op == "random_search":
        _, s["tasks"], s["offs"] = _groups(case, seed)
    elif op == "proposal":
        _, s["tasks"], s["offs"] = _groups(case, seed)
        s["net"] = _surrogate(case, seed, 65536)
    else:
        b, gid, orders, _, T = _training_batch(case, seed)
        s.update(tasks=_dev(b.tasks), offs=_dev(b.offs), gid=_dev(gid), orders=_dev(orders), T=_dev(T),
                 net=_surrogate(case, seed, case["rows"]))
    return s


def run(s):
    op = s["op"]
    if op == "group":
        summary, _ = tgo.exhaustive(s["tasks"], s["model"])
        orders, ns = tgo.heuristic(s["tasks"], s["offs"], s["model"])
        return {"summary": summary, "order": orders, "ns": ns}
    if op == "per_order":
        summary, times = tgo.exhaustive(s["tasks"], s["model"], per_order=True)
        return {"summary": summary, "times": times}
    if op == "batch":
        return s["plan"].run(s["tasks"], s["offs"])
    if op == "evaluate":
        return tgo.evaluate(s["tasks"], s["orders"], s["model"])
    if op == "memory":
        return tgo.exhaustive_mem(s["tasks"], s["mem"], s["capacity"], s["model"])[0]
    if op == "concurrent":
        return tgo.exhaustive_cke(s["tasks"], s["units"], s["case"]["capacity"], s["model"])[0]
    if op == "rounds":
        summary, _, groups = tgo.rounds(s["tasks"], s["case"]["workers"], s["case"]["rounds"], s["model"])
        return {"summary": summary, "groups": groups}
    if op == "random_search":
        return tgo.random_search(s["tasks"], s["offs"], s["case"]["samples"], s["seed"])
    if op == "proposal":
        return s["net"].search(s["tasks"], s["offs"], s["case"]["samples"], 64, s["seed"])
    grad, loss = s["net"].grad(s["tasks"], s["offs"], s["orders"], s["gid"], s["T"])
    return {"grad": grad, "loss": loss}


def _nodes(n):
    """Distinct non-empty prefixes of the orderings of n tasks: each is placed once."""
    return sum(math.factorial(n) // math.factorial(n - j) for j in range(1, n + 1))


def work(case):
    """Bytes of the inputs and outputs; operations: 32-bit integer ones, 16 per
    placed task (one DMA engine: 5) and 10 per ordering for the reduction, 100
    per drawn ordering; floating-point ones of the network."""
    op = case["op"]
    place = 16 if case.get("engines", 2) == 2 else 5
    if op in ("group", "per_order", "memory", "concurrent"):
        n = case["n"]
        f = math.factorial(n)
        return {"bytes": 24 * n + 136 + (8 * f if op == "per_order" else 0), "flops": place * _nodes(n) + 10 * f}
    if op == "rounds":
        w, r = case["workers"], case["rounds"]
        f = math.factorial(w)
        return {"bytes": 24 * w * r + 136, "flops": place * _nodes(w) * sum(f ** i for i in range(r)) + 10 * f ** r}
    if op == "evaluate":
        return {"bytes": case["rows"] * (case["n"] + 8), "flops": case["rows"] * case["n"] * place}
    mean = (case["n_lo"] + case["n_hi"]) / 2
    if op == "batch":
        sizes = range(case["n_lo"], case["n_hi"] + 1)
        per = sum(place * _nodes(n) + 10 * math.factorial(n) for n in sizes) / len(sizes)
        return {"bytes": case["groups"] * (24 * mean + 140), "flops": case["groups"] * per}
    if op == "grad":
        return {"bytes": case["rows"] * 28 + 4 * 2 * 144385, "flops": case["rows"] * 836096}
    per = 100 + 16 * mean if op == "random_search" else 287232
    return {"bytes": case["groups"] * (24 * mean + 68), "flops": case["groups"] * case["samples"] * per}


def exact(case, seed):
    if case["op"] != "grad":
        return None  # whole numbers and packed records
    b, gid, orders, lb, T = _training_batch(case, seed)
    at = "cuda" if torch.cuda.is_available() else "cpu"
    live = orders != 255
    row = b.offs[gid].astype(np.int64)[:, None] + np.where(live, orders, 0)
    f = np.log1p(b.tasks[row] / 1e3) / math.log1p(20000.0) * live[:, :, None]
    x = torch.as_tensor(f.reshape(len(gid), 48)).to(at)
    y = torch.as_tensor(T / lb[gid] - 1.0).to(at)
    w = [torch.as_tensor(v.astype(np.float64)).to(at).requires_grad_() for v in _weights(seed)]
    for i in (0, 2, 4):
        x = torch.relu(x @ w[i].t() + w[i + 1])
    loss = ((x @ w[6] + w[7] - y) ** 2).mean()
    g = torch.autograd.grad(loss, w)
    return {"grad": torch.cat([v.reshape(-1) for v in g]), "loss": loss.detach().reshape(1)}
