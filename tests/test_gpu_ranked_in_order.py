"""Ranked positions of snapshots that come in queue order, formed by the kernel for queue order: runs of equal deadlines inside a
lane's four requests, over lanes, over blocks of 256 and to the end of a snapshot, at the edges of the capacities and off 16-byte
boundaries; marked and unmarked snapshots in one batch; snapshots that end anywhere in a workgroup laid out for a larger bound."""
import dataclasses

import numpy as np
import pytest

from paper_2602_08747_amd import workloads as wl

pytestmark = pytest.mark.gpu
I32 = np.iinfo(np.int32)


def in_order(seed, sizes, S, runs, shuffle=()):
    """Snapshots of the given sizes in deadline order; a deadline is shared by about `runs` neighbours (0: by all)."""
    K = len(sizes)
    w = wl.random_workload(seed, K=K, S=S, n_per_snapshot=4, modes=(wl.MODE_LBF,))
    rng = np.random.default_rng([seed, 5])
    ptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(ptr[-1])
    deadline = np.empty(n, np.int64)
    for u in range(K):
        m = sizes[u]
        steps = rng.random(m) < (1.0 / runs if runs else 0.0)
        deadline[ptr[u]:ptr[u + 1]] = 20000 + np.cumsum(steps * rng.integers(1, 40, m))
        if u in shuffle:
            rng.shuffle(deadline[ptr[u]:ptr[u + 1]])
    return dataclasses.replace(w, arrival=np.zeros(n, np.int32), deadline=deadline.astype(np.int32),
                               stage=rng.integers(0, S, n).astype(np.int32), snap_ptr=ptr, now=rng.integers(0, 30000, K).astype(np.int32))


def wide(w):
    d = w.deadline.copy()
    for u in range(w.K):
        lo, hi = w.snap_ptr[u], w.snap_ptr[u + 1]
        d[lo:hi][: max(1, (hi - lo) // 3)] = I32.min
        d[lo:hi][-max(1, (hi - lo) // 4):] = I32.max
    return dataclasses.replace(w, deadline=d)


EDGES = {"1024": [513, 1023, 1024, 1, 0, 700] * 3, "2048": [2048, 1025, 2045, 3] * 3, "4096": [4096, 4095, 2049] * 2,
         "8192": [8192, 4097, 8189, 8191]}


@pytest.mark.parametrize("S", [2, 3, 6])
@pytest.mark.parametrize("runs", [0, 1, 2, 5, 90, 600])
@pytest.mark.parametrize("edge", list(EDGES))
def test_ranked_in_order(oracle_mod, edge, runs, S):
    check(oracle_mod, in_order(100 * runs + S, EDGES[edge], S, runs))


@pytest.mark.parametrize("which", ["wide", "some-shuffled", "many-small"])
def test_ranked_in_order_mixed(oracle_mod, which):
    if which == "wide":
        w = wide(in_order(1, [3000, 8192, 5001], 5, 3))
    elif which == "some-shuffled":
        w = in_order(2, [2500, 4096, 3333, 4001], 4, 2, shuffle=(1, 3))
    else:
        w = in_order(3, [600 + i for i in range(300)], 6, 4, shuffle=tuple(range(0, 300, 7)))
    check(oracle_mod, w)


ENDS = [255, 256, 257, 1, 0, 3, 511, 513, 767, 1023, 1025, 1279, 1793]


@pytest.mark.parametrize("S", [2, 5])
@pytest.mark.parametrize("runs", [0, 1, 3, 200])
@pytest.mark.parametrize("sizes,bound", [(ENDS, 2048), (ENDS, 4096), (ENDS, 8192), ([2049, 2047, 1021, 3071], 8192), ([1024] * 9, 4096),
                                         ([1025] * 9, 8192), ([1365] * 260, 4096), ([1366] * 260, 4096), ([2730] * 260, 8192), ([2731] * 259 + [2732], 8192)])
def test_loose_bound(oracle_mod, sizes, bound, runs, S):
    """A bound far above the sizes, on both sides of the mean size from which the in-order kernel forms the ranked estimates itself
    (1024 of few snapshots, a third of the workgroup's capacity of many, where that is 4096 or 8192)."""
    times = 1 if len(sizes) > 100 else -(-8300 // sum(sizes))          # (calls of at most 8192 requests don't come here)
    w = in_order(1000 * runs + S + bound, sizes * times, S, runs)
    if runs != 1:
        w = wide(w)
    check(oracle_mod, w, bound)


@pytest.mark.parametrize("S", [2, 3, 4, 6])
@pytest.mark.parametrize("B,W,quotient", [(1, 256, (1 << 17) - 1), (1, 1, 1 << 16), (2, 255, (1 << 17) - 1), (64, 256, (1 << 17) - 1)])
def test_sums_past_32_bits(oracle_mod, B, W, quotient, S):
    """A chain whose first queue holds nearly all requests, its waits at the top of the short form (8000 batches near 2^30), and whose later stages take
    up to 2^31 - 1 for a batch that is not full: along the first queue the sums cross 2^32 (INT32_MAX with one later stage)."""
    sizes = [8192, 6001, 8000, 2049]
    rng = np.random.default_rng([B, W, S])
    w = in_order(S, sizes, S, 3)
    row_ptr, col = wl.csr_from_edges(S, wl.chain_edges(S))
    batch, workers = np.full(S, 64, np.int32), np.full(S, 3, np.int32)
    batch[0], workers[0] = B, W
    full = W * quotient + W - 1
    lat = np.full((S, 64), 1000, np.int64)                # (a full batch of the later stages; the table falls)
    lat[0] = full - (np.maximum(B - 1 - np.arange(64), 0) * full) // 100
    whole = (1 << 32 if S > 2 else 1 << 31) - 4000 // B * quotient
    lat[1:, :63] = whole // (S - 1)
    stage, d = [], []
    for m in sizes:
        k = np.zeros(m, np.int32)
        k[rng.permutation(m)[:40 * (S - 1)]] = np.repeat(np.arange(1, S), 40)
        stage.append(k)
        d.append(np.sort(rng.integers(I32.min, I32.max, m, endpoint=True)))
    d[0][:400], d[0][-300:] = I32.min, I32.max
    w = dataclasses.replace(w, dag_shared=1, dag_row_ptr=row_ptr, dag_col=col, batch=batch, workers=workers,
                            lat_us=np.ascontiguousarray(lat.reshape(-1), np.int32), order_mode=np.full(S, wl.MODE_LBF, np.int32),
                            deadline=np.concatenate(d).astype(np.int32), stage=np.concatenate(stage), now=np.array([I32.min, 0, I32.max, I32.min], np.int32))
    assert lat.max() <= I32.max and full // W < 1 << 17
    check(oracle_mod, w)


def check(oracle_mod, w, bound=None):
    """Against the oracle, and the marks behind the workspace's 256-byte header: 0 where the in-order kernel took a snapshot."""
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libpard.so")
    from paper_2602_08747_amd import binding
    ref = oracle_mod.run(w, threads=8, ranked=True)
    s = binding.Session(w, max_snapshot_requests=bound)
    s.workspace[64:64 + w.K] = -5
    s.est.fill_(-3)
    s.drop.fill_(7)
    s.estimate_drop(ranked=True)
    marks = s.workspace[64:64 + w.K].cpu().numpy()
    falls = [bool((np.diff(w.deadline[w.snap_ptr[u]:w.snap_ptr[u + 1]].astype(np.int64)) < 0).any()) for u in range(w.K)]
    assert np.array_equal(marks, np.array(falls, np.int32))
    s.compact()
    got = s.results()
    for k in ("est", "drop", "order", "seg_ptr", "surv_idx", "surv_ptr"):
        assert np.array_equal(got[k], ref[k]), k
    assert s.status_word() == 0
