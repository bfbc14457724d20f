"""GPU parity: libpard (through its C-ABI) against the CPU oracle, bit for bit.

Integer microseconds throughout, so every output must be identical: est, drop, order,
seg_ptr, surv_idx, surv_ptr.
"""
import numpy as np
import pytest

from paper_2602_08747_amd import workloads as wl

pytestmark = pytest.mark.gpu

INT32_MAX = 2**31 - 1
KEYS = ("est", "drop", "order", "seg_ptr", "surv_idx", "surv_ptr")
FORCE_SORT = 1 << 20        # promised snapshot bound above the on-chip capacity -> radix-sort path


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libpard.so")
    from paper_2602_08747_amd import binding
    binding.load_library()
    return binding


def check(gpu, oracle_mod, w, max_snap=None, threads=8):
    print(f"case {w.name} n={w.n} K={w.K} S={w.S} max_snap={max_snap}", flush=True)
    ref = oracle_mod.run(w, threads=threads)
    s = gpu.Session(w, max_snapshot_requests=max_snap)
    s.run()
    got = s.results()
    for k in KEYS:
        if not np.array_equal(got[k], ref[k]):
            bad = np.flatnonzero(got[k] != ref[k]) if got[k].shape == ref[k].shape else None
            raise AssertionError(f"{w.name}: {k} differs (shape {got[k].shape} vs {ref[k].shape}); "
                                 f"first bad {None if bad is None else bad[:8]}; "
                                 f"got {None if bad is None else got[k][bad[:8]]} want {None if bad is None else ref[k][bad[:8]]}")
    assert s.status_word() == 0
    # the whole path in one call leaves the same outputs
    for t in (s.est, s.drop, s.order, s.seg_ptr, s.surv_idx, s.surv_ptr):
        t.fill_(0x55)
    s.run_one_call()
    got = s.results()
    for k in KEYS:
        assert np.array_equal(got[k], ref[k]), (w.name, "one call", k)
    assert s.status_word() == 0
    return s, ref


# ---- the five benchmark configurations at full size --------------------------------------

@pytest.mark.parametrize("cfg", [1, 2, 3, 4, 5])
def test_full_config(gpu, oracle_mod, cfg):
    w = wl.make_workload(cfg)
    check(gpu, oracle_mod, w)


@pytest.mark.parametrize("cfg,kw", [(1, {}), (2, dict(n_requests=300001)), (3, dict(n_requests=250007)),
                                     (4, dict(n_requests=700003)), (5, dict(n_snapshots=97, per_snapshot=8192))])
def test_config_shapes_permuted(gpu, oracle_mod, cfg, kw):
    """Same shapes, request order shuffled (arrival-ordered input is nearly sorted), mixed drop masks."""
    w = wl.make_workload(cfg, permute=True, **kw)
    w.now[:] = np.maximum(0, w.now.astype(np.int64) - 280000).astype(np.int32)
    if cfg in (2, 3, 4):
        w.lat_us[:] = np.maximum(1, w.lat_us // 400)       # out of deep overload: some requests survive
    s, ref = check(gpu, oracle_mod, w)
    assert 0 < ref["drop"].mean() < 1


@pytest.mark.parametrize("n,permute", [(1 << 20, True), (None, False), (None, True)])
def test_config4_half_survivors(gpu, oracle_mod, n, permute):
    """Bursty DAG with an SLO of half the arrival span (a labelled variant, not one of the five configurations):
    compaction with roughly half the queue surviving and estimates below the saturation value, at one million
    requests and at the configuration's full 16.8 million, in arrival order and shuffled."""
    w = wl.half_survivors(wl.make_workload(4, n_requests=n, permute=permute))
    s, ref = check(gpu, oracle_mod, w, threads=16)
    assert 0.1 < ref["drop"].mean() < 0.9
    assert (ref["est"] < INT32_MAX).mean() > 0.5


def test_large_path_beyond_two_to_the_25(gpu, oracle_mod):
    """More than 2^25 requests in one snapshot: beyond the 1024 ranges of 2^15 request ids through which the results
    of smaller calls go back to request order, so every result is written at its request's place by a kernel of its
    own and unpacked by a streaming one.  Configuration 4's shape, shuffled, with a mixed drop mask."""
    w = wl.half_survivors(wl.make_workload(4, n_requests=(1 << 25) + 4097, permute=True))
    s, ref = check(gpu, oracle_mod, w, threads=16)
    assert 0.1 < ref["drop"].mean() < 0.9


def test_large_path_beyond_64_chunks(gpu, oracle_mod):
    """More than 2^24 requests in one snapshot: the radix passes then scan their chunk totals in a kernel of
    their own (up to 128 chunks every chunk workgroup scans them itself), and the results go back to request order
    through more than 512 ranges of request ids (two ranges to a thread in the last pass).  Configuration 4's shape,
    shuffled, with latencies scaled so that the drop mask is mixed."""
    w = wl.half_survivors(wl.make_workload(4, n_requests=(1 << 24) + 8193, permute=True))
    s, ref = check(gpu, oracle_mod, w, threads=16)
    assert 0.1 < ref["drop"].mean() < 0.9


# ---- both kernel paths on the same small inputs -------------------------------------------

@pytest.mark.parametrize("seed", range(12))
def test_random_small_both_paths(gpu, oracle_mod, seed):
    K = 1 + (seed * 5) % 7
    S = 1 + (seed * 3) % 9
    w = wl.random_workload(100 + seed, K=K, S=S, n_per_snapshot=50 + 37 * seed, monotone=(seed % 2 == 0),
                           tie_heavy=(seed % 3 == 2))
    check(gpu, oracle_mod, w)
    check(gpu, oracle_mod, w, max_snap=FORCE_SORT)


@pytest.mark.parametrize("mode", [wl.MODE_LBF, wl.MODE_HBF, wl.MODE_FCFS, None])
def test_order_modes(gpu, oracle_mod, mode):
    w = wl.make_workload(5, n_snapshots=9, per_snapshot=5000, permute=True, order_mode=mode)
    if mode is None:
        w.order_mode[:] = np.arange(w.order_mode.size) % 3          # mixed per stage
    w.deadline[::5] = w.deadline[1::5][: w.deadline[::5].size]      # plenty of equal keys
    check(gpu, oracle_mod, w)
    check(gpu, oracle_mod, w, max_snap=FORCE_SORT)


@pytest.mark.parametrize("m", [0, 1, 2, 63, 64, 65, 4095, 8191, 8192])
def test_snapshot_sizes_on_chip(gpu, oracle_mod, m):
    w = wl.make_workload(5, n_snapshots=3, per_snapshot=m, permute=True)
    check(gpu, oracle_mod, w)


@pytest.mark.parametrize("per", [1, 31, 64, 65, 100, 127, 128])
def test_one_wave_per_snapshot(gpu, oracle_mod, per):
    """Promised bounds up to 128 requests take the path that gives a snapshot to a single wave (64 or 128
    sorted in registers): snapshots that fill the wave exactly or not, ragged mixes with empty ones, every
    order mode and heavy ties, own and shared DAGs, few and many stages, the downstream latency given
    from outside, and the same snapshots under a larger promise (the workgroup path)."""
    for permute in (True, False):
        w = wl.make_workload(5, n_snapshots=9, per_snapshot=per, permute=permute)
        check(gpu, oracle_mod, w)
        check(gpu, oracle_mod, w, max_snap=128)
        check(gpu, oracle_mod, w, max_snap=256)
        check(gpu, oracle_mod, w, max_snap=512)
    half = max(per // 2, 1)
    for i, kw in enumerate((dict(S=5, dag_shared=0), dict(S=8, dag_shared=1), dict(S=9, dag_shared=0, tie_heavy=True),
                            dict(S=12, dag_shared=1), dict(S=3, dag_shared=0, modes=(wl.MODE_FCFS,)),
                            dict(S=4, dag_shared=1, modes=(wl.MODE_HBF,), tie_heavy=True))):
        for attempt in range(20):           # a random DAG of a dozen stages may expand to more paths than a plan takes
            w = wl.random_workload(9000 + 10 * per + i + 1000 * attempt, K=41, n_per_snapshot=half, **kw)
            rows = w.dag_row_ptr.reshape(-1, w.S + 1)
            cols = np.split(w.dag_col, np.cumsum(rows[:, -1])[:-1])
            if max(wl.count_paths_any_order(w.S, rows[d], cols[d]) * w.S for d in range(len(rows))) <= 4096:
                break
        assert w.max_snapshot_requests <= 128
        s, ref = check(gpu, oracle_mod, w)
        rng = np.random.default_rng(per + i)
        sub = rng.integers(0, 60_000, size=w.K * w.S).astype(np.int64)
        want = oracle_mod.run(w, threads=8, sub=sub)
        import torch
        s.run(sub=torch.from_numpy(sub).to(s.dev))
        got = s.results()
        for k in KEYS:
            assert np.array_equal(got[k], want[k]), (per, i, k)
        # sequentially consistent dropping, with modest downstream latencies so that queues are cut in the middle
        for given in (None, sub // 8):
            want = oracle_mod.run(w, threads=8, sub=given, consistent=True)
            s.run(sub=None if given is None else torch.from_numpy(given).to(s.dev), consistent=True)
            got = s.results()
            for k in KEYS:
                assert np.array_equal(got[k], want[k]), (per, i, "consistent", given is None, k)


def test_one_wave_per_snapshot_many_snapshots(gpu, oracle_mod):
    w = wl.make_workload(5, n_snapshots=20000, per_snapshot=61, permute=True)
    _, ref = check(gpu, oracle_mod, w, threads=16)
    assert 0 < ref["drop"].mean() < 1
    w = wl.random_workload(31337, K=3000, S=6, n_per_snapshot=64, dag_shared=0)
    assert w.max_snapshot_requests <= 128
    s, _ = check(gpu, oracle_mod, w, threads=16)
    plain = s.results()
    want = oracle_mod.run(w, threads=16, consistent=True)
    s.run(consistent=True)
    got = s.results()
    for k in KEYS:
        assert np.array_equal(got[k], want[k]), k
    assert not np.array_equal(got["drop"], plain["drop"])          # the variant is not vacuous on this input


@pytest.mark.parametrize("mix", ["uniform", "mostly-small", "geometric", "all-empty", "steps"])
def test_mixed_snapshot_sizes(gpu, oracle_mod, mix):
    """Batches whose snapshots differ widely in size under one promise (the workgroup of a call is sized for the
    largest): snapshots that end before some of a thread's request groups, empty ones, sizes at every capacity step."""
    import torch
    K = 700
    rng = np.random.default_rng(sum(map(ord, mix)))
    base = wl.make_workload(5, n_snapshots=K, per_snapshot=8192, permute=True)
    sizes = {"uniform": rng.integers(0, 8193, K),
             "mostly-small": np.where(rng.random(K) < 0.9, rng.integers(0, 257, K), rng.integers(4000, 8193, K)),
             "geometric": np.minimum(rng.geometric(1 / 600, K), 8192),
             "all-empty": np.zeros(K, np.int64),
             "steps": rng.choice([0, 1, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192], K)}[mix]
    w = wl.with_snapshot_sizes(base, sizes)
    for max_snap in (None, 8192, 5000, 9000):          # 9000: the large-snapshot path
        if max_snap is not None and max_snap < w.max_snapshot_requests:
            continue
        s, ref = check(gpu, oracle_mod, w, max_snap=max_snap)
        sub = rng.integers(0, 300_000, size=w.K * w.S).astype(np.int64)
        for given, consistent in ((sub, False), (None, True), (sub // 16, True)):
            want = oracle_mod.run(w, threads=8, sub=given, consistent=consistent)
            s.run(sub=None if given is None else torch.from_numpy(given).to(s.dev), consistent=consistent)
            got = s.results()
            for k in KEYS:
                assert np.array_equal(got[k], want[k]), (mix, max_snap, given is None, consistent, k)
            assert s.status_word() == 0


@pytest.mark.parametrize("cap", [256, 512, 1024, 2048, 4096, 8192])
def test_every_workgroup_capacity(gpu, oracle_mod, cap):
    """The on-chip kernel comes in several capacities, picked from the promised snapshot bound: snapshots that
    fill a capacity exactly (the path without bounds tests), fall one short of it, or mix sizes below it; the
    same snapshots under a larger promise (a larger workgroup) must give the same result."""
    for per, permute in ((cap, True), (cap, False), (cap - 1, True), (cap // 2 + 3, True)):
        w = wl.make_workload(5, n_snapshots=5, per_snapshot=per, permute=permute)
        check(gpu, oracle_mod, w)
        if cap < 8192:
            check(gpu, oracle_mod, w, max_snap=2 * cap)
    # ragged sizes up to cap; each capacity has variants for pipelines of at most 8, at most 16 and more stages
    for S in (7, 8, 9, 13, 16, 17):
        for attempt in range(40):           # a random DAG of many stages may expand to more paths than a plan takes
            w = wl.random_workload(600 + cap + S + 1000 * attempt, K=9, S=S, n_per_snapshot=cap // 2,
                                   dag_shared=0 if S < 16 else 1)
            rows = w.dag_row_ptr.reshape(-1, w.S + 1)
            cols = np.split(w.dag_col, np.cumsum(rows[:, -1])[:-1])
            if max(wl.count_paths_any_order(w.S, rows[d], cols[d]) * w.S for d in range(len(rows))) <= 4096:
                break
        assert w.max_snapshot_requests <= cap
        check(gpu, oracle_mod, w, max_snap=cap)
        ref = oracle_mod.run(w, threads=8, consistent=True)
        s = gpu.Session(w, max_snapshot_requests=cap)
        s.run(consistent=True)
        got = s.results()
        for k in KEYS:
            assert np.array_equal(got[k], ref[k]), (cap, S, k)


@pytest.mark.parametrize("K,cap", [(2049, 512), (1025, 1024), (513, 2048), (257, 4096), (257, 8192)])
def test_every_workgroup_capacity_of_large_batches(gpu, oracle_mod, K, cap):
    """The few snapshots above take wide workgroups; one snapshot more than those serve (1024 threads per compute unit, 256 of
    them) takes sixteen requests a thread: full to the capacity and one short, in order and not, sequentially consistent, and
    pipelines of 12 and of 17 stages."""
    for per, permute in ((cap, True), (cap, False), (cap - 1, True)):
        check(gpu, oracle_mod, wl.make_workload(5, n_snapshots=K, per_snapshot=per, permute=permute), max_snap=cap)
    for S in (6, 12, 17):
        w = wl.random_workload(700 + cap, K=K, S=S, n_per_snapshot=cap, dag_shared=1, vary_sizes=False, time_span=20 * cap,
                               slo_choices=(3 * cap, 6 * cap))
        w.lat_us[:] = np.maximum(1, w.lat_us // 20)
        rng = np.random.default_rng(cap)
        w = wl.with_snapshot_sizes(w, np.where(np.arange(K) % 3 == 2, rng.integers(0, cap + 1, K), cap))
        s, ref = check(gpu, oracle_mod, w, max_snap=cap)
        assert 0 < ref["drop"].mean() < 1
        ref = oracle_mod.run(w, threads=8, consistent=True)
        s.run(consistent=True)
        got = s.results()
        for k in KEYS:
            assert np.array_equal(got[k], ref[k]), (cap, S, k)


@pytest.mark.parametrize("per", [40, 700, 1500, 3000, 8000])
def test_sixty_four_stages(gpu, oracle_mod, per):
    """The largest stage count: a chain of 64 stages plus a few shortcuts, every workgroup capacity, both paths."""
    S, K = 64, 4
    rng = np.random.default_rng(6400 + per)
    rp, col = wl.csr_from_edges(S, wl.chain_edges(S) + [(3, 40), (10, 63), (20, 51)])
    sizes = rng.integers(per // 2, per + 1, size=K)
    snap_ptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(snap_ptr[-1])
    arrival = rng.integers(0, 200_000, n).astype(np.int32)
    w = wl.Workload(name=f"chain64-{per}", K=K, S=S, dag_shared=1, dag_row_ptr=rp, dag_col=col,
                    batch=rng.integers(1, 65, S).astype(np.int32), workers=rng.integers(1, 9, S).astype(np.int32),
                    lat_us=np.ascontiguousarray(wl.monotone_tables(rng, S).reshape(-1) // 20, np.int32),
                    order_mode=rng.integers(0, 3, S).astype(np.int32), arrival=arrival,
                    deadline=(arrival + rng.choice([100_000, 900_000, 4_000_000], n)).astype(np.int32),
                    stage=rng.integers(0, S, n).astype(np.int32), snap_ptr=snap_ptr,
                    now=np.full(K, 150_000, np.int32))
    _, ref = check(gpu, oracle_mod, w)
    assert 0.02 < ref["drop"].mean() < 0.98, ref["drop"].mean()
    check(gpu, oracle_mod, w, max_snap=FORCE_SORT)
    for max_snap in (None, FORCE_SORT):
        ref = oracle_mod.run(w, threads=8, consistent=True)
        s = gpu.Session(w, max_snapshot_requests=max_snap)
        s.run(consistent=True)
        got = s.results()
        for k in KEYS:
            assert np.array_equal(got[k], ref[k]), (per, max_snap, k)


@pytest.mark.parametrize("n", [0, 1, 2, 255, 4096, 4097, 8193, 12289, 70001])
def test_sizes_sort_path(gpu, oracle_mod, n):
    w = wl.make_workload(3, n_requests=n, permute=True)
    check(gpu, oracle_mod, w, max_snap=FORCE_SORT)


@pytest.mark.parametrize("n,what", [((1 << 22) + 12345, "large tiles, a ragged last tile and a ragged last range of request ids"),
                                    (1 << 22, "the largest request count on small tiles"),
                                    ((1 << 21) + 2049, "small tiles, ranges of 2^13 ids"),
                                    ((1 << 20) - 3, "ranges of 2^11 ids, the last one short")])
def test_sort_path_tile_and_range_steps(gpu, oracle_mod, n, what):
    """Request counts on either side of the steps the radix passes take (tiles of 2048 or 4096 elements; the way
    back to request order through ranges of 2^11 to 2^15 request ids), shuffled, with a mixed drop mask."""
    w = wl.half_survivors(wl.make_workload(4, n_requests=n, permute=True))
    s, ref = check(gpu, oracle_mod, w, threads=16)
    assert 0.1 < ref["drop"].mean() < 0.9, what


def test_many_queues_sort_path(gpu, oracle_mod):
    """More queues (snapshots x stages) than the large-snapshot path keeps on chip per workgroup."""
    w = wl.random_workload(31, K=12, S=8, n_per_snapshot=700, dag_shared=0)
    assert w.K * w.S > 64
    check(gpu, oracle_mod, w, max_snap=FORCE_SORT)


def test_many_large_snapshots(gpu, oracle_mod):
    """So many snapshots above the on-chip size that global request index and queue id no longer fit
    one 32-bit word together: the large-snapshot path carries the index inside the snapshot instead."""
    w = wl.make_workload(5, n_snapshots=300, per_snapshot=9000, permute=True)
    w.now[:] = np.maximum(0, w.now.astype(np.int64) - 250000).astype(np.int32)
    assert (w.n - 1).bit_length() + (w.K * w.S - 1).bit_length() > 32
    s, ref = check(gpu, oracle_mod, w, threads=16)
    assert 0 < ref["drop"].mean() < 1


def test_snapshot_larger_than_promised_on_the_large_path(gpu):
    w = wl.make_workload(5, n_snapshots=3, per_snapshot=20000)
    s = gpu.Session(w, max_snapshot_requests=9000)
    s.run()
    s.results()
    assert s.status_word() & 1


def test_ragged_multi_snapshot_large(gpu, oracle_mod):
    """Several snapshots of very different sizes, some above the on-chip capacity, own DAG each."""
    w = wl.random_workload(7, K=5, S=6, n_per_snapshot=9000, dag_shared=0, time_span=2_000_000,
                           slo_choices=(150000, 400000))
    assert w.max_snapshot_requests > 8192
    check(gpu, oracle_mod, w)


# ---- degenerate inputs -------------------------------------------------------------------

def test_all_ties_single_stage(gpu, oracle_mod):
    w = wl.make_workload(1, n_requests=8192)
    w.deadline[:] = 123456
    w.stage[:] = 1
    check(gpu, oracle_mod, w)
    check(gpu, oracle_mod, w, max_snap=FORCE_SORT)


def test_clustered_keys(gpu, oracle_mod):
    """Half of the keys equal, the rest spread over the whole int32 range (worst case for bucketing)."""
    w = wl.make_workload(2, n_requests=6000, permute=True)
    w.deadline[::2] = 77
    w.deadline[1::4] = INT32_MAX
    w.deadline[3::8] = 0
    check(gpu, oracle_mod, w)
    check(gpu, oracle_mod, w, max_snap=FORCE_SORT)


def test_extreme_values(gpu, oracle_mod):
    """INT32_MAX deadlines are never dropped; huge latencies saturate; negative times are ordered correctly."""
    w = wl.make_workload(3, n_requests=5000, permute=True)
    w.lat_us[:] = INT32_MAX
    w.deadline[1::7] = -5
    w.deadline[::3] = INT32_MAX
    w.arrival[::2] = -100
    w.now[:] = INT32_MAX
    s, ref = check(gpu, oracle_mod, w)
    assert not ref["drop"][::3].any() and (ref["est"] == INT32_MAX).all()
    check(gpu, oracle_mod, w, max_snap=FORCE_SORT)
    w.now[:] = -(2**31)
    check(gpu, oracle_mod, w)


def test_batch_and_worker_extremes(gpu, oracle_mod):
    for B, W in ((1, 1), (64, 1), (1, 1 << 20), (63, 7), (64, 16), (3, 1000)):
        w = wl.make_workload(2, n_requests=7000, permute=True)
        w.batch[:] = B
        w.workers[:] = W
        w.now[:] = 0
        check(gpu, oracle_mod, w)
    w = wl.make_workload(2, n_requests=9000, permute=True)
    w.batch[:] = [1, 64, 5, 33, 2]
    w.workers[:] = [1 << 20, 1, 3, 1, 999]
    w.lat_us[:] = (w.lat_us.astype(np.int64) * 5000).clip(0, INT32_MAX).astype(np.int32)    # wait term beyond 32 bits
    check(gpu, oracle_mod, w, max_snap=FORCE_SORT)
    check(gpu, oracle_mod, w, max_snap=FORCE_SORT)


def test_out_of_range_stage_is_clamped(gpu, oracle_mod):
    w = wl.make_workload(1, n_requests=3000)
    w.stage[::11] = -7
    w.stage[5::13] = 1000
    check(gpu, oracle_mod, w)
    check(gpu, oracle_mod, w, max_snap=FORCE_SORT)


def test_many_paths_dag(gpu, oracle_mod):
    """Six diamonds in series: 64 paths, 13-stage paths."""
    S = 19
    edges = []
    for d in range(6):
        a = 3 * d
        edges += [(a, a + 1), (a, a + 2), (a + 1, a + 3), (a + 2, a + 3)]
    rp, cl = wl.csr_from_edges(S, edges)
    w = wl.make_workload(4, n_requests=6000, permute=True)
    rng = np.random.default_rng(1)
    w2 = wl.Workload(name="diamonds", K=1, S=S, dag_shared=1, dag_row_ptr=rp, dag_col=cl,
                     batch=rng.integers(1, 65, S).astype(np.int32), workers=rng.integers(1, 9, S).astype(np.int32),
                     lat_us=wl.monotone_tables(rng, S).reshape(-1), order_mode=np.zeros(S, np.int32),
                     arrival=w.arrival, deadline=w.deadline, stage=rng.integers(0, S, w.n).astype(np.int32),
                     snap_ptr=w.snap_ptr, now=w.now)
    assert gpu.pard_plan_check(1, S, 1, rp, cl, w2.batch, w2.workers, w2.lat_us, w2.order_mode)[1] == 64
    check(gpu, oracle_mod, w2)
    check(gpu, oracle_mod, w2, max_snap=FORCE_SORT)


# ---- API behaviour ------------------------------------------------------------------------

@pytest.mark.parametrize("max_snap", [None, FORCE_SORT])
def test_compact_with_arbitrary_masks(gpu, oracle_mod, max_snap):
    """pard_compact is a function of (order, seg_ptr, drop) alone; per-snapshot and streamed compaction."""
    import torch
    w = wl.make_workload(5, n_snapshots=11, per_snapshot=4099, permute=True)
    s, ref = check(gpu, oracle_mod, w, max_snap=max_snap)
    rng = np.random.default_rng(9)
    for p in (0.0, 1.0, 0.5, 0.03):
        mask = ((rng.random(w.n) < p) * rng.integers(1, 256, w.n)).astype(np.uint8)     # any nonzero byte drops
        s.drop.copy_(torch.from_numpy(mask).to(s.dev))
        s.compact()
        got = s.results()
        want_idx, want_ptr = oracle_mod.compact(w.K, w.S, ref["order"], ref["seg_ptr"], mask)
        assert np.array_equal(got["surv_ptr"], want_ptr) and np.array_equal(got["surv_idx"], want_idx)


@pytest.mark.parametrize("cfg,kw", [(5, dict(n_snapshots=7, per_snapshot=8192)), (5, dict(n_snapshots=5, per_snapshot=5000)),
                                     (4, dict(n_requests=150001))])
@pytest.mark.parametrize("max_snap", [None, FORCE_SORT])
def test_compact_unaligned_buffers(gpu, oracle_mod, cfg, kw, max_snap):
    """Buffers that start at odd byte offsets (views into larger allocations) give the same survivors."""
    import torch
    w = wl.make_workload(cfg, permute=True, **kw)
    s, ref = check(gpu, oracle_mod, w, max_snap=max_snap)
    rng = np.random.default_rng(21)
    mask = (rng.random(w.n) < 0.4).astype(np.uint8)
    want_idx, want_ptr = oracle_mod.compact(w.K, w.S, ref["order"], ref["seg_ptr"], mask)
    n = w.n
    for off_drop, off_idx in ((3, 1), (13, 3), (16, 2)):
        drop_big = torch.ones(n + 64, dtype=torch.uint8, device=s.dev)
        drop = drop_big[off_drop:off_drop + n]
        drop.copy_(torch.from_numpy(mask).to(s.dev))
        order_big = torch.zeros(n + 16, dtype=torch.int32, device=s.dev)
        order = order_big[off_idx:off_idx + n]
        order.copy_(s.order)
        surv_big = torch.full((n + 16,), -7, dtype=torch.int32, device=s.dev)
        surv = surv_big[off_idx:off_idx + n]
        gpu.pard_compact(s.plan, n, s.max_snap, order, s.seg_ptr, drop, surv, s.surv_ptr, s.workspace)
        torch.cuda.synchronize()
        got_ptr = s.surv_ptr.cpu().numpy()
        assert np.array_equal(got_ptr, want_ptr)
        assert np.array_equal(surv.cpu().numpy()[:want_ptr[-1]], want_idx)
        sb = surv_big.cpu().numpy()
        assert (sb[:off_idx] == -7).all() and (sb[off_idx + want_ptr[-1]:] == -7).all()   # nothing written outside


@pytest.mark.parametrize("shape", ["wave", "workgroup-small", "workgroup-full", "workgroup-ragged", "sorted"])
def test_estimate_unaligned_buffers(gpu, oracle_mod, shape):
    """Request arrays and outputs that start at odd offsets (views into larger allocations): the 16-byte accesses
    of every kernel path fall back or shift, the results stay the same and nothing is written outside the views."""
    import torch
    if shape == "wave":
        w = wl.make_workload(5, n_snapshots=300, per_snapshot=61, permute=True)
    elif shape == "workgroup-small":
        w = wl.make_workload(5, n_snapshots=40, per_snapshot=700, permute=True)
    elif shape == "workgroup-full":
        w = wl.make_workload(5, n_snapshots=6, per_snapshot=8192, permute=True)
    elif shape == "workgroup-ragged":
        w = wl.with_snapshot_sizes(wl.make_workload(5, n_snapshots=30, per_snapshot=8192, permute=True),
                                   np.random.default_rng(3).integers(0, 8193, 30))
    else:
        w = wl.make_workload(3, n_requests=90_001, permute=True)
    s, ref = check(gpu, oracle_mod, w)
    want_c = oracle_mod.run(w, threads=8, consistent=True)
    n = w.n
    for o32, o8 in ((1, 1), (2, 6), (3, 3), (4, 16)):
        def view32(src):
            big = torch.full((n + 32,), -7, dtype=torch.int32, device=s.dev)
            v = big[o32:o32 + n]
            if src is not None:
                v.copy_(src)
            return big, v
        _, arrival = view32(s.arrival)
        _, deadline = view32(s.deadline)
        _, stage = view32(s.stage)
        est_big, est = view32(None)
        order_big, order = view32(None)
        drop_big = torch.full((n + 64,), 9, dtype=torch.uint8, device=s.dev)
        drop = drop_big[o8:o8 + n]
        for consistent, want in ((False, ref), (True, want_c)):
            if consistent:
                gpu.pard_estimate_drop_consistent(s.plan, n, s.max_snap, arrival, deadline, stage, s.snap_ptr, s.now, None,
                                                  est, drop, order, s.seg_ptr, s.workspace)
            else:
                gpu.pard_estimate_drop(s.plan, n, s.max_snap, arrival, deadline, stage, s.snap_ptr, s.now,
                                       est, drop, order, s.seg_ptr, s.workspace)
            torch.cuda.synchronize()
            assert np.array_equal(est.cpu().numpy(), want["est"]), (shape, o32, consistent)
            assert np.array_equal(drop.cpu().numpy(), want["drop"]), (shape, o8, consistent)
            assert np.array_equal(order.cpu().numpy(), want["order"]), (shape, o32, consistent)
            assert np.array_equal(s.seg_ptr.cpu().numpy(), want["seg_ptr"]), (shape, consistent)
            for big, off in ((est_big, o32), (order_big, o32)):
                h = big.cpu().numpy()
                assert (h[:off] == -7).all() and (h[off + n:] == -7).all()
            h = drop_big.cpu().numpy()
            assert (h[:o8] == 9).all() and (h[o8 + n:] == 9).all()
        assert s.status_word() == 0


@pytest.mark.parametrize("case", ["on-chip", "sorted", "sorted-consistent", "on-chip-ranked"])
def test_graph_capture_and_replay(gpu, oracle_mod, case):
    """The hot calls only enqueue kernels (no allocation, no synchronisation, no memset nodes), so they can be
    recorded into a HIP graph.  Every replay, with different inputs in the same buffers and eager work in
    between, must match the oracle."""
    import torch
    if case.startswith("on-chip"):
        w = wl.make_workload(5, n_snapshots=12, per_snapshot=6000, permute=True)
    else:
        w = wl.make_workload(3, n_requests=120_000, permute=True)
    consistent, ranked = case.endswith("consistent"), case.endswith("ranked")
    s = gpu.Session(w)
    s.run(consistent=consistent, ranked=ranked)                 # warm up outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        s.run(consistent=consistent, ranked=ranked)
    base_now = w.now.copy()
    for shift in (0, -150_000, -400_000, 0):
        w.now[:] = np.maximum(-2**31, base_now.astype(np.int64) + shift).astype(np.int32)
        s.now.copy_(torch.from_numpy(w.now).to(s.dev))
        s.est.zero_(); s.drop.zero_(); s.order.zero_(); s.surv_idx.zero_()      # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = s.results()
        ref = oracle_mod.run(w, threads=8, consistent=consistent, ranked=ranked)
        for k in KEYS:
            assert np.array_equal(got[k], ref[k]), (case, shift, k)
        assert s.status_word() == 0


def test_repeatable_and_stream(gpu, oracle_mod):
    import torch
    w = wl.make_workload(4, n_requests=300000, permute=True)
    s, ref = check(gpu, oracle_mod, w)
    side = torch.cuda.Stream()
    for _ in range(3):
        s.est.zero_(); s.order.zero_(); s.surv_idx.zero_()
        side.wait_stream(torch.cuda.current_stream())
        s.run(stream=side)
        side.synchronize()
        got = s.results()
        for k in KEYS:
            assert np.array_equal(got[k], ref[k])


def test_snapshot_larger_than_promised_sets_status(gpu, oracle_mod):
    w = wl.make_workload(5, n_snapshots=4, per_snapshot=500)
    s = gpu.Session(w, max_snapshot_requests=100)
    s.run()
    s.results()
    assert s.status_word() & 1


def test_error_codes_with_device(gpu):
    import torch
    w = wl.make_workload(1)
    s = gpu.Session(w)
    tiny = torch.zeros(64, dtype=torch.int32, device=s.dev)
    assert gpu.pard_estimate_drop(s.plan, s.n, s.max_snap, s.arrival, s.deadline, s.stage, s.snap_ptr, s.now, s.est,
                                  s.drop, s.order, s.seg_ptr, tiny, check=False) == -8
    assert gpu.pard_estimate_drop(s.plan, -1, s.max_snap, s.arrival, s.deadline, s.stage, s.snap_ptr, s.now, s.est,
                                  s.drop, s.order, s.seg_ptr, s.workspace, check=False) == -2
    assert gpu.pard_estimate_drop(s.plan, s.n, s.max_snap, s.arrival, None, s.stage, s.snap_ptr, s.now, s.est,
                                  s.drop, s.order, s.seg_ptr, s.workspace, check=False) == -1
    assert gpu.pard_compact(s.plan, s.n, s.max_snap, s.order, s.seg_ptr, s.drop, s.surv_idx, s.surv_ptr, tiny[:8], check=False) == -8
    assert gpu.pard_plan_info(s.plan) == (1, 3)


def test_streamed_compaction_shares_the_device(gpu, oracle_mod):
    """No kernel of the streamed compaction waits for another workgroup, so such calls may run next to each other and
    next to other work: two sessions compact on two streams at the same time, several times over, while a third
    stream keeps the compute units busy; every result is the oracle's."""
    import torch
    cases = []
    for seed, n in ((0, 3_000_001), (1, 1_700_003)):
        w = wl.make_workload(4, n_requests=n, permute=True, seed=seed)
        w.lat_us[:] = np.maximum(1, w.lat_us // 400)
        w.now[:] = np.maximum(0, w.now.astype(np.int64) - 280000).astype(np.int32)
        s, ref = check(gpu, oracle_mod, w)
        cases.append((s, ref, torch.cuda.Stream()))
    busy = torch.cuda.Stream()
    filler = torch.zeros(64 << 20, dtype=torch.float32, device=cases[0][0].dev)
    torch.cuda.synchronize()
    for _ in range(5):
        for s, _, st in cases:
            s.surv_idx.fill_(-7)
            s.surv_ptr.fill_(-7)
        torch.cuda.synchronize()
        with torch.cuda.stream(busy):
            for _ in range(8):
                filler.mul_(1.0001).add_(1.0)
        for s, _, st in cases:
            s.compact(stream=st)
        torch.cuda.synchronize()
        for s, ref, _ in cases:
            got = s.results()
            assert np.array_equal(got["surv_ptr"], ref["surv_ptr"]) and np.array_equal(got["surv_idx"], ref["surv_idx"])
            assert s.status_word() == 0


@pytest.mark.parametrize("permute", [True, False])
def test_hundred_repeats_are_identical(gpu, oracle_mod, permute):
    """Configuration 5 at full size, a hundred runs of the whole path (through the two calls and through the one call
    in turn): every output of every run is bit for bit the first run's, which is the oracle's."""
    import torch
    w = wl.make_workload(5, permute=permute)
    s, ref = check(gpu, oracle_mod, w, threads=16)
    names = ("est", "drop", "order", "seg_ptr", "surv_idx", "surv_ptr")
    total = int(ref["surv_ptr"][-1])
    want = {k: getattr(s, k).clone() for k in names}
    for i in range(100):
        for k in names:
            getattr(s, k).fill_(0x33)
        if i % 2:
            s.run_one_call()
        else:
            s.run()
        for k in names:
            a, b = getattr(s, k), want[k]
            if k == "surv_idx":
                a, b = a[:total], b[:total]
            assert torch.equal(a, b), (i, k)
    assert s.status_word() == 0
