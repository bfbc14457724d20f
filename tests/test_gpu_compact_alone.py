"""pard_compact where one workgroup takes all queue slots, at the edges of that rule (slots in all, queues, the promised bound),
and the move of staged survivors on both sides of its step."""
import numpy as np
import pytest

from paper_2602_08747_amd import workloads as wl

pytestmark = pytest.mark.gpu
KEYS = ("est", "drop", "order", "seg_ptr", "surv_idx", "surv_ptr")


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libpard.so")
    from paper_2602_08747_amd import binding
    binding.load_library()
    return binding


def mixed(seed, K, S, per, **kw):
    """Latencies small enough that a part of every queue survives."""
    w = wl.random_workload(seed, K=K, S=S, n_per_snapshot=per, time_span=20 * per, slo_choices=(10 * per, 30 * per), **kw)
    w.lat_us[:] = np.maximum(1, w.lat_us // (100 if per < 2000 else 30))
    return w


def agree(gpu, oracle_mod, w, max_snap=None, one_call=False):
    ref = oracle_mod.run(w, threads=8)
    s = gpu.Session(w, max_snapshot_requests=max_snap)
    s.surv_idx.fill_(-9)
    s.run_one_call() if one_call else s.run()
    got = s.results()
    for k in KEYS:
        assert np.array_equal(got[k], ref[k]), k
    assert (s.surv_idx[len(ref["surv_idx"]):w.n].cpu().numpy() == -9).all()       # nothing behind the survivors
    assert s.status_word() == 0


@pytest.mark.parametrize("n", [1, 3, 1023, 4096, 4097, 8191, 8192, 8193])
@pytest.mark.parametrize("max_snap", [None, 1 << 16])
def test_one_snapshot(gpu, oracle_mod, n, max_snap):
    w = mixed(n, 1, 5, n, vary_sizes=False)
    agree(gpu, oracle_mod, w, max_snap)


@pytest.mark.parametrize("K,S,per", [(7, 6, 500), (1365, 3, 2), (1366, 3, 2), (2, 4, 2500), (3, 10, 2000), (100, 5, 81)])
def test_several_snapshots(gpu, oracle_mod, K, S, per):
    """1365 x 3 queues and one more than the rule takes; bounds above 2048 are compacted snapshot by snapshot."""
    w = mixed(K + S, K, S, per, dag_shared=1)
    agree(gpu, oracle_mod, w)


@pytest.mark.parametrize("per", [4095, 4097, 8192])
def test_staged_survivors_move(gpu, oracle_mod, per):
    w = wl.half_survivors(wl.make_workload(5, n_snapshots=9, per_snapshot=per, permute=True))
    agree(gpu, oracle_mod, w, one_call=True)


@pytest.mark.parametrize("per,bound", [(40, 8192), (1024, 4096), (1025, 4096), (2048, 8192), (2049, 2049), (2049, 8192), (4096, 4096), (4097, 8192)])
@pytest.mark.parametrize("K", [3, 1100])
def test_staged_survivors_move_by_mean_size(gpu, oracle_mod, per, bound, K):
    """One wave, four or eight move a snapshot's survivors, by the mean size beside the promised bound; at least four of few snapshots."""
    w = mixed(per, K, 4, per, dag_shared=1, vary_sizes=False)
    agree(gpu, oracle_mod, w, bound, one_call=True)


def test_broken_promise_is_reported(gpu):
    """A single snapshot larger than the promised per-snapshot bound's workgroup holds: flagged, nothing written out of place."""
    import torch
    w = wl.random_workload(3, K=1, S=3, n_per_snapshot=5000, vary_sizes=False)
    s = gpu.Session(w)
    s.run()
    torch.cuda.synchronize()
    assert s.status_word() == 0
    gpu.pard_compact(s.plan, s.n, 3000, s.order, s.seg_ptr, s.drop, s.surv_idx, s.surv_ptr, s.workspace)
    torch.cuda.synchronize()
    assert s.status_word() == 1
