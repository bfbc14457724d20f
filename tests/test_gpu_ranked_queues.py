"""Ranked positions on chip at the edges of their dispatch: snapshot sizes around the steps of the workgroup, 16 and 17 stages,
stages without the short cost form, ties, deadlines over the whole int32 range, arrival order among the queues."""
import dataclasses

import numpy as np
import pytest

from paper_2602_08747_amd import workloads as wl

pytestmark = pytest.mark.gpu
I32 = np.iinfo(np.int32)


def case(seed, K, S, requests, **kw):
    return wl.random_workload(seed, K=K, S=S, n_per_snapshot=requests, **kw)


def wide(w, seed):
    """Deadlines over all of int32, the ends among them."""
    rng = np.random.default_rng(seed)
    d = rng.integers(I32.min, I32.max, w.n, endpoint=True).astype(np.int32)
    d[:: max(1, w.n // 5)] = I32.max
    d[1:: max(1, w.n // 7)] = I32.min
    return dataclasses.replace(w, name=w.name + "-wide", deadline=d)


CASES = {
    "tiny": lambda: case(1, 40, 3, 3, modes=(wl.MODE_LBF,)),
    "128": lambda: case(2, 5, 6, 128, modes=(wl.MODE_LBF,), vary_sizes=False),
    "129-hbf": lambda: case(3, 5, 6, 129, modes=(wl.MODE_HBF,), vary_sizes=False),
    "513-16-stages": lambda: case(4, 3, 16, 513, vary_sizes=False),
    "17-stages": lambda: case(5, 3, 17, 300),
    "2049-mixed-orders": lambda: case(6, 2, 8, 2049, vary_sizes=False),
    "8192-ties": lambda: case(7, 2, 5, 8192, tie_heavy=True, vary_sizes=False),
    "slow-stages": lambda: dataclasses.replace(case(8, 4, 7, 700), workers=np.full(4 * 7, 300, np.int32), dag_shared=0)
    if case(8, 4, 7, 700).dag_shared == 0 else dataclasses.replace(case(8, 4, 7, 700), workers=np.full(7, 300, np.int32)),
    "wide": lambda: wide(case(9, 3, 6, 900, modes=(wl.MODE_LBF, wl.MODE_HBF)), 9),
    "one-outlier": lambda: outlier(case(10, 2, 4, 3000, modes=(wl.MODE_LBF,))),
    "one-outlier-hbf": lambda: outlier(case(11, 3, 3, 700, modes=(wl.MODE_HBF,))),
    "whole-rows": lambda: alternating(case(12, 3, 2, 256, modes=(wl.MODE_LBF,), vary_sizes=False)),
    "whole-rows-outlier": lambda: outlier(alternating(case(13, 3, 2, 2048, modes=(wl.MODE_LBF,), vary_sizes=False))),
    "one-stage": lambda: case(14, 5, 1, 700),
    "one-stage-wave": lambda: case(15, 50, 1, 40),
    "one-stage-large": lambda: case(16, 2, 1, 9000, vary_sizes=False),
    "two-slow-stages-200": lambda: slow(case(17, 9, 2, 100)),
    "two-slow-stages-700": lambda: slow(case(18, 4, 2, 700, vary_sizes=False)),
    "eight-slow-stages-4000": lambda: slow(case(19, 2, 8, 4000, vary_sizes=False)),
    "nine-slow-stages": lambda: slow(case(20, 2, 9, 600, vary_sizes=False)),
}


def slow(w):
    """More workers than the short cost form covers."""
    return dataclasses.replace(w, workers=np.full_like(w.workers, 300))


def alternating(w):
    """Queues of whole rows of 64 slots."""
    return dataclasses.replace(w, stage=(np.arange(w.n) % w.S).astype(np.int32))


def outlier(w):
    d = w.deadline.copy()
    d[w.n // 2] = I32.max - 1                       # all others fall into one bucket
    return dataclasses.replace(w, deadline=d)


@pytest.mark.parametrize("which", list(CASES))
def test_ranked_on_chip(oracle_mod, which):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libpard.so")
    from paper_2602_08747_amd import binding
    w = CASES[which]()
    ref = oracle_mod.run(w, threads=8, ranked=True)
    s = binding.Session(w)
    s.run(ranked=True)
    got = s.results()
    for k in ("est", "drop", "order", "seg_ptr", "surv_idx", "surv_ptr"):
        assert np.array_equal(got[k], ref[k]), k
