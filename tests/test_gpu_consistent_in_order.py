"""Sequentially consistent dropping on snapshots in queue order and around them: the closed count of positions in time against
a plain count on the CPU, and both on-chip kernels against the oracle at the edges of their rule."""
import dataclasses

import numpy as np
import pytest

from paper_2602_08747_amd import workloads as wl

I32 = np.iinfo(np.int32)


def cost(pos, B, W, lat):
    pos = np.asarray(pos, np.int64)
    return -(-pos // B) * lat[B - 1] // W + lat[np.minimum(pos + 1, B) - 1]


def positions_in_time(budget, B, W, lat):
    """The kernel's closed form, in float32 where it uses floats (short-queue waits: exact there, so integers here)."""
    if budget < lat[0]:
        return 0
    b = min(budget, 2**32 - 1)
    wait = lambda q: q * lat[B - 1] // W  # noqa: E731
    full, first = int(lat[B - 1]), int(wait(1))
    if b < full or b - full < first:
        if b < first:
            return 1
        return 1 + int(np.searchsorted(lat[1:B], b - first, side="right"))
    inv = np.float32(W) / np.float32(full) if full > 0 else np.float32(1e30)
    with np.errstate(over="ignore"):
        q = int(min((np.float32(b - full) + np.float32(1.0)) * inv, np.float32(8190.0)))
    if wait(q) > b - full:
        q -= 1
    elif wait(q + 1) <= b - full:
        q += 1
    return q * B + 1


@pytest.mark.parametrize("seed", range(60))
def test_positions_in_time_is_a_count(seed):
    """Against counting positions 0 .. 8191 one by one, at budgets on both sides of every kind of step."""
    rng = np.random.default_rng(seed)
    B, W = int(rng.integers(1, 65)), int(rng.choice([1, 2, 3, 7, 16, 255, 256]))
    scale = int(rng.choice([1, 3, 50, 3000, 200_000]))
    lat = np.cumsum(rng.integers(0, scale + 1, 64)).astype(np.int64)
    lat = np.minimum(lat, 2**31 - 1)
    if lat[B - 1] // W >= 1 << 17:
        lat //= int(lat[B - 1] // W >> 17) + 2
    every = cost(np.arange(8192), B, W, lat)
    budgets = np.concatenate([every[rng.integers(0, 8192, 200)][:, None] + np.array([-1, 0, 1])[None], every[:3 * B].reshape(-1, 1) + np.array([-1, 0, 1])], axis=None)
    budgets = np.concatenate([budgets, rng.integers(-5, 2**31 + 2**31 - 1, 50), [-(2**40), 2**32, 2**40]])
    for budget in budgets.tolist():
        assert min(positions_in_time(budget, B, W, lat), 8192) == int(np.searchsorted(every, budget, side="right")), (budget, B, W, seed)


def queued(seed, K, S, per, relax=20, **kw):
    w = wl.random_workload(seed, K=K, S=S, n_per_snapshot=per, time_span=20 * per, slo_choices=(3 * per,), modes=(wl.MODE_LBF,), **kw)
    w.lat_us[:] = np.maximum(0, w.lat_us // relax)
    return wl.in_deadline_order(w)


def extremes(w):
    d = w.deadline.copy()
    for u in range(w.K):
        lo, hi = int(w.snap_ptr[u]), int(w.snap_ptr[u + 1])
        if hi - lo > 20:
            d[lo:lo + 5] = I32.min
            d[hi - 7:hi] = I32.max                 # never dropped
    return dataclasses.replace(w, deadline=d)


def falling(w):
    w.lat_us[:] = w.lat_us[::-1].copy()           # tables that fall: no closed form
    return w


CASES = {
    "4097": lambda: queued(1, 3, 6, 4097, vary_sizes=False),
    "4096": lambda: queued(2, 3, 6, 4096, vary_sizes=False),
    "8192-one-stage": lambda: queued(3, 2, 1, 8192, vary_sizes=False),
    "ragged": lambda: queued(4, 9, 5, 4200),
    "overload": lambda: queued(5, 3, 4, 8000, relax=3, vary_sizes=False),
    "extremes": lambda: extremes(queued(6, 2, 3, 8191, vary_sizes=False)),
    "ties": lambda: wl.in_deadline_order(wl.random_workload(7, K=2, S=4, n_per_snapshot=5000, tie_heavy=True, modes=(wl.MODE_LBF,), vary_sizes=False)),
    "zero-latencies": lambda: queued(8, 2, 3, 5000, relax=1 << 30, vary_sizes=False),
    "falling-tables": lambda: falling(queued(9, 2, 5, 5000, vary_sizes=False)),
    "seven-stages": lambda: queued(10, 2, 7, 6000, vary_sizes=False),
    "not-in-order": lambda: wl.random_workload(11, K=3, S=6, n_per_snapshot=6000, time_span=120_000, modes=(wl.MODE_LBF,), slo_choices=(60_000, 200_000, 400_000)),
    "high-budget": lambda: wl.random_workload(12, K=2, S=6, n_per_snapshot=6000, time_span=120_000, modes=(wl.MODE_HBF,), slo_choices=(200_000, 900_000)),
    "slow-stages": lambda: slow(queued(13, 2, 4, 5000, vary_sizes=False)),
}


def slow(w):
    return dataclasses.replace(w, workers=np.full_like(w.workers, 300))


@pytest.mark.gpu
@pytest.mark.parametrize("which", list(CASES))
def test_consistent_on_chip(oracle_mod, which):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libpard.so")
    from paper_2602_08747_amd import binding
    w = CASES[which]()
    ref = oracle_mod.run(w, threads=8, consistent=True)
    s = binding.Session(w)
    s.run(consistent=True)
    got = s.results()
    for k in ("est", "drop", "order", "seg_ptr", "surv_idx", "surv_ptr"):
        assert np.array_equal(got[k], ref[k]), k
