"""The potential form's transcription in opcount.py gives the oracle's times, in walks
and across rates, so the operations it counts are those of the method."""
import math

import numpy as np

import opcount
from oracle import model as M
from paper_1806_10113_amd import workloads as W


def test_walks_equal_the_oracle():
    rng = np.random.default_rng(4)
    for q_log2, p_h, p_d in ((2, 3, 3), (0, 1, 1), (2, 1, 4), (3, 5, 7), (4, 15, 9)):
        r, model = opcount.Rates(q_log2, p_h, p_d), M.Model(1 << q_log2, p_h, p_d)
        if p_h == 1 << q_log2:
            continue  # the form needs p_htd < q
        for tasks in (W.single_group_mixed(12, 1), rng.integers(0, 40, size=(9, 3)), rng.integers(0, 3, size=(7, 3))):
            n = len(tasks)
            for sub in rng.choice(math.factorial(n) // 120, size=3, replace=False):
                ts = opcount.walk_subtree(tasks.tolist(), int(sub), 5, r, opcount.Counter(), form="potential")
                want = [M.simulate(tasks.tolist(), M.nth_permutation(n, int(sub) * 120 + l), model) for l in range(120)]
                assert ts == want, (n, sub, q_log2, p_h, p_d)


def test_windows_are_the_chain_forms():
    a, b = opcount.Counter(), opcount.Counter()
    opcount.walk_subtree(W.single_group_mixed(12, 1), 4321, 5, opcount.Rates(), a)
    opcount.walk_subtree(W.single_group_mixed(12, 1), 4321, 5, opcount.Rates(), b, form="potential")
    assert a.windows == b.windows and b.ops > 0
