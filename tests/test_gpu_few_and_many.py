"""On-chip kernels on both sides of the rule that gives few snapshots wide workgroups (threads times snapshots against 1024 per compute
unit: 256 of them on this device), in queue order and not, for every capacity and every kind of call."""
import dataclasses

import numpy as np
import pytest

from paper_2602_08747_amd import workloads as wl

pytestmark = pytest.mark.gpu
KEYS = ("est", "drop", "order", "seg_ptr", "surv_idx", "surv_ptr")

SHAPES = [(2, 300), (2048, 270), (2049, 270), (3, 1000), (1024, 530), (1025, 530), (5, 2000), (512, 1030), (513, 1030), (4, 4096), (256, 2050),
          (257, 2050), (3, 8192), (256, 4100), (257, 4100)]


def snapshots(K, per, kind):
    w = wl.random_workload(K + per, K=K, S=6 if kind != "many-stages" else 17, n_per_snapshot=per, time_span=20 * per, slo_choices=(4 * per,) if kind == "in-order" else (3 * per, 6 * per),
                           modes={"high": (wl.MODE_HBF,), "any": (wl.MODE_LBF, wl.MODE_HBF, wl.MODE_FCFS)}.get(kind, (wl.MODE_LBF,)),
                           dag_shared=1, vary_sizes=False, tie_heavy=False)
    w.lat_us[:] = np.maximum(1, w.lat_us // 20)
    rng = np.random.default_rng(per)
    w = wl.with_snapshot_sizes(w, np.where(np.arange(K) % 4 == 2, rng.integers(0, per + 1, K), per))
    if kind == "in-order":
        w = wl.in_deadline_order(w)
    return w


@pytest.mark.parametrize("K,per", SHAPES)
@pytest.mark.parametrize("kind", ["in-order", "low", "high", "any"])
def test_few_and_many(oracle_mod, K, per, kind):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libpard.so")
    from paper_2602_08747_amd import binding
    w = snapshots(K, per, kind)
    s = binding.Session(w, max_snapshot_requests=per)
    for call in ("two", "one", "consistent"):
        if call != "one":
            ref = oracle_mod.run(w, threads=8, consistent=call == "consistent")
        s.run_one_call() if call == "one" else s.run(consistent=call == "consistent")
        got = s.results()
        for k in KEYS:
            assert np.array_equal(got[k], ref[k]), (call, k)
    assert s.status_word() == 0


@pytest.mark.parametrize("per,bound", [(1024, 4096), (1025, 4096), (2048, 8192), (2049, 8192), (100, 8192), (30, 300), (128, 512), (129, 512), (256, 1024), (257, 1024), (512, 2048), (513, 2048)])
@pytest.mark.parametrize("kind", ["in-order", "low", "high"])
def test_few_under_a_loose_bound(oracle_mod, per, bound, kind):
    """Snapshots around a quarter of the capacity."""
    from paper_2602_08747_amd import binding
    w = wl.random_workload(per, K=9, S=3, n_per_snapshot=per, time_span=20 * per, slo_choices=(4 * per,) if kind == "in-order" else (3 * per, 6 * per),
                           modes=(wl.MODE_HBF,) if kind == "high" else (wl.MODE_LBF,), dag_shared=1, vary_sizes=False)
    w.lat_us[:] = np.maximum(1, w.lat_us // 20)
    if kind == "in-order":
        w = wl.in_deadline_order(w)
    s = binding.Session(w, max_snapshot_requests=bound)
    for consistent in (False, True):
        ref = oracle_mod.run(w, threads=8, consistent=consistent)
        s.run(consistent=consistent)
        got = s.results()
        for k in KEYS:
            assert np.array_equal(got[k], ref[k]), (consistent, k)
    assert s.status_word() == 0


@pytest.mark.parametrize("K,per", [(2, 500), (3, 4000), (2, 8192), (300, 2100)])
def test_many_stages(oracle_mod, K, per):
    from paper_2602_08747_amd import binding
    w = snapshots(K, per, "many-stages")
    ref = oracle_mod.run(w, threads=8)
    s = binding.Session(w, max_snapshot_requests=per)
    s.run()
    got = s.results()
    for k in KEYS:
        assert np.array_equal(got[k], ref[k]), k


@pytest.mark.parametrize("K,most,size", [(2, 1500, 1700), (600, 1500, 1700), (2, 5000, 6000), (300, 5000, 5100)])
def test_larger_than_promised(K, most, size):
    """Flagged, and the others are right, with wide workgroups and without."""
    import torch
    from paper_2602_08747_amd import binding
    w = wl.random_workload(K, K=K, S=5, n_per_snapshot=most, modes=(wl.MODE_LBF,), dag_shared=1, vary_sizes=False)
    s = binding.Session(w, max_snapshot_requests=most)
    s.run()
    good = s.results()
    assert s.status_word() == 0
    short = most - (size - most)                           # the first snapshot grows into the second
    s.snap_ptr[1] = size
    s.run()
    torch.cuda.synchronize()
    assert s.status_word() == 1 and short > 0
    lo = int(w.snap_ptr[2])
    if K > 2:
        assert np.array_equal(s.est.cpu().numpy()[lo:], good["est"][lo:]) and np.array_equal(s.drop.cpu().numpy()[lo:], good["drop"][lo:])


@pytest.mark.parametrize("times", [1, 130])                # wide workgroups, and the usual ones
@pytest.mark.parametrize("most,size", [(300, 307), (1000, 1013), (1500, 1700), (3000, 4001), (5000, 6000)])
@pytest.mark.parametrize("kind", ["in-order", "low", "high"])
def test_ranked_larger_than_promised(oracle_mod, most, size, kind, times):
    """Ranked calls leave the plain estimates to no one else: a snapshot larger than promised still gets those of its first requests, the
    last one, whose queues end where the promise does, the ranked ones, and the others are right."""
    import torch
    from paper_2602_08747_amd import binding
    sizes = [most, size, most - 7] * times + [size]
    K, lasts = len(sizes), len(sizes) - 1
    w = wl.random_workload(most, K=K, S=3, n_per_snapshot=size, time_span=20 * most, slo_choices=(4 * most,) if kind == "in-order" else (3 * most, 6 * most),
                           modes=(wl.MODE_HBF,) if kind == "high" else (wl.MODE_LBF,), dag_shared=1, vary_sizes=False)
    row_ptr, col = wl.csr_from_edges(3, wl.chain_edges(3))
    w = dataclasses.replace(w, dag_row_ptr=row_ptr, dag_col=col, lat_us=np.maximum(1, w.lat_us // 20).astype(np.int32))
    w = wl.with_snapshot_sizes(w, sizes)
    if kind == "in-order":
        w = wl.in_deadline_order(w)
    served = wl.with_snapshot_sizes(w, np.minimum(sizes, most))
    plain, ranked = oracle_mod.run(served, threads=8), oracle_mod.run(served, threads=8, ranked=True)
    assert not np.array_equal(plain["est"], ranked["est"])
    s = binding.Session(w, max_snapshot_requests=most)
    s.est.fill_(-3)
    s.drop.fill_(7)
    s.estimate_drop(ranked=True)
    torch.cuda.synchronize()
    assert s.status_word() == 1
    est, drop = s.est.cpu().numpy(), s.drop.cpu().numpy()
    for u in range(K):
        a, b = int(w.snap_ptr[u]), int(served.snap_ptr[u])
        m = min(sizes[u], most)
        want = plain if sizes[u] > most and u != lasts else ranked
        assert np.array_equal(est[a:a + m], want["est"][b:b + m]) and np.array_equal(drop[a:a + m], want["drop"][b:b + m]), u
        assert (est[a + m:a + sizes[u]] == -3).all() and (drop[a + m:a + sizes[u]] == 7).all()
