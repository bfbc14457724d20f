"""Sequentially consistent dropping where the chains of all queues are one prefix minimum: empty queues, one queue, 64 queues,
sizes at the edges of the workgroup, off 16-byte boundaries, and a snapshot with one queue that has to be walked instead."""
import dataclasses

import numpy as np
import pytest

from paper_2602_08747_amd import workloads as wl

pytestmark = pytest.mark.gpu


def case(seed, sizes, S, ordered, skip=()):
    K = len(sizes)
    w = wl.random_workload(seed, K=K, S=S, n_per_snapshot=4, modes=(wl.MODE_LBF,), dag_shared=0 if K > 1 else 1)
    if S > 16:                                      # few paths: the oracle follows every one
        row_ptr, col = wl.csr_from_edges(S, wl.chain_edges(S))
        w = dataclasses.replace(w, dag_shared=1, dag_row_ptr=row_ptr, dag_col=col, batch=w.batch[:S], workers=w.workers[:S],
                                lat_us=w.lat_us[:S * wl.LAT_ENTRIES], order_mode=w.order_mode[:S])
    rng = np.random.default_rng([seed, 9])
    ptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(ptr[-1])
    deadline = rng.integers(0, 3_000_000, n).astype(np.int32)
    deadline[:: 17] = np.iinfo(np.int32).max
    if ordered:
        for u in range(K):
            deadline[ptr[u]:ptr[u + 1]].sort()
    used = np.setdiff1d(np.arange(S), skip)
    return dataclasses.replace(w, arrival=np.zeros(n, np.int32), deadline=deadline, stage=rng.choice(used, n).astype(np.int32),
                               snap_ptr=ptr, now=rng.integers(0, 200_000, K).astype(np.int32), lat_us=np.maximum(1, w.lat_us // 3).astype(np.int32))


@pytest.mark.parametrize("ordered", [False, True])
@pytest.mark.parametrize("S,skip", [(1, ()), (3, (0,)), (6, (1, 2, 5)), (6, ()), (64, (0, 17, 63))])
@pytest.mark.parametrize("sizes", [[8192] * 2, [4097, 8191, 3001, 8189, 2050], [8192, 7, 5000, 6001, 1, 8000] + [4100] * 300])
def test_all_chains_at_once(oracle_mod, sizes, S, skip, ordered):
    check(oracle_mod, case(sum(sizes) % 1000 + S, sizes, S, ordered, skip))


@pytest.mark.parametrize("ordered", [False, True])
def test_one_queue_walked(oracle_mod, ordered):
    w = case(5, [8000, 4444, 8192], 5, ordered)
    w.batch[2] = 8
    w.lat_us.reshape(-1, 64)[2, :8] = [90, 80, 70, 60, 50, 40, 30, 20]      # the cost falls with the position
    check(oracle_mod, w)


def check(oracle_mod, w):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libpard.so")
    from paper_2602_08747_amd import binding
    ref = oracle_mod.run(w, threads=8, consistent=True)
    s = binding.Session(w)
    s.run(consistent=True)
    got = s.results()
    for k in ("est", "drop", "order", "seg_ptr", "surv_idx", "surv_ptr"):
        assert np.array_equal(got[k], ref[k]), k
