"""The sampled batch-wait quantile where paths are evaluated by the set of their stages (pipelines of at most 8 stages):
the float form of a wait against integers on the CPU, and the kernel against the oracle at the edges of its dispatch."""
import numpy as np
import pytest

from paper_2602_08747_amd import workloads as wl


def test_wait_in_floats_is_exact():
    """(-a) mod d as q*d - a with q = floor(fma(a, 1/d, 1/2)), one correction: every a < 2^31, 2^10 <= d < 2^24.
    The product of two float32 values and the added half are exact in float64, so rounding that once is the fused sum."""
    rng = np.random.default_rng(3)
    ds = np.unique(np.concatenate([np.arange(1024, 1100), 2 ** np.arange(10, 24), 2 ** np.arange(11, 25) - 1, 3 ** np.arange(7, 15),
                                   rng.integers(1024, 1 << 24, 400)]))
    for d in ds[(ds >= 1024) & (ds < 1 << 24)]:
        top = (2**31 - 1) // d
        k = np.unique(np.concatenate([np.arange(0, 50), top - np.arange(0, 50), rng.integers(0, top + 1, 2000)]))
        a = (k[k >= 0][:, None] * d + np.array([-1, 0, 1, d // 2, d - d // 2])[None, :]).ravel()
        a = np.concatenate([a[(a >= 0) & (a < 2**31)], rng.integers(0, 2**31, 2000)]).astype(np.int64)
        rcp = np.float32(1.0) / np.float32(d)
        z = (a.astype(np.float32).astype(np.float64) * np.float64(rcp) + 0.5).astype(np.float32)
        q = z.astype(np.int64)
        assert q.max() < 1 << 24
        v = ((q * d - a) & 0xFFFFFFFF).astype(np.uint64)
        w = np.minimum(v, (v + np.uint64(d)) & np.uint64(0xFFFFFFFF))
        assert np.array_equal(w.astype(np.int64), (-a) % d), d


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libpard.so")
    from paper_2602_08747_amd import binding
    binding.load_library()
    return binding


CASES = [
    # K, S, requests, shared, latency scale (numerator, denominator), samples, lambda
    (1, 1, 50, 1, (1, 1), 100, (1, 2)),                     # nothing downstream
    (3000, 1, 4, 1, (1, 1), 100, (1, 2)),                   # nor in many snapshots
    (2, 8, 300, 1, (1, 1), 2047, (1, 10)),                  # few path entries: path by path
    (300, 8, 40, 1, (1, 1), 2047, (1, 10)),                 # a few workgroups per snapshot; one below a block of samples
    (250, 8, 30, 0, (1, 400), 2048, (1, 2048)),              # durations below 2^10: the integer form; the smallest total
    (700, 5, 30, 0, (400, 1), 2049, (2048, 2049)),          # durations around 2^24; next to the largest total
    (1030, 4, 4, 0, (1, 1), 1, (1, 2)),                     # one workgroup per snapshot; one sample
    (1025, 6, 5, 1, (1, 30), 4097, (9, 10)),                # durations on both sides of 2^10
    (2, 9, 300, 0, (1, 1), 2049, (1, 10)),                  # nine stages: path by path
    (1100, 3, 4, 1, (1, 1), 50, (1, 10)),                   # a wave takes 256 samples at a time: a part of one wave's,
    (900, 4, 4, 0, (1, 30), 255, (1, 2)),                   # all but one,
    (900, 4, 4, 0, (1, 1), 256, (255, 256)),                # all,
    (1030, 4, 4, 0, (1, 30), 257, (1, 10)),                 # one into the next wave's,
    (700, 5, 4, 0, (1, 1), 16384, (1, 10)),                 # the most samples there may be
]


@pytest.mark.gpu
@pytest.mark.parametrize("K,S,requests,shared,scale,M,lam", CASES)
def test_sampled_quantile_by_stage_set(gpu, oracle_mod, K, S, requests, shared, scale, M, lam):
    import torch
    w = wl.random_workload(100 * S + K, K=K, S=S, n_per_snapshot=requests, dag_shared=shared)
    w.lat_us[:] = np.minimum(w.lat_us.astype(np.int64) * scale[0] // scale[1], 1 << 25)
    s = gpu.Session(w)
    rng = np.random.default_rng(M)
    samples = rng.integers(-5, 2**31 - 1, M).astype(np.int32)
    picks = rng.integers(0, 2**32, M * S, dtype=np.uint64).astype(np.uint32)
    qlen = np.concatenate([np.bincount(np.clip(w.stage[w.snap_ptr[u]:w.snap_ptr[u + 1]], 0, S - 1), minlength=S)
                           for u in range(K)]).astype(np.int32)
    got = s.planner(gpu.SUB_FULL, lam, torch.from_numpy(samples).to(s.dev), torch.from_numpy(picks.view(np.int32)).to(s.dev))
    torch.cuda.synchronize()
    assert np.array_equal(s.qlen.cpu().numpy(), qlen)
    for qdelay in (None, rng.integers(-10, 100_000, K * S).astype(np.int32)):
        if qdelay is not None:
            s.sub.fill_(-7)
            got = s.planner(gpu.SUB_FULL, lam, torch.from_numpy(samples).to(s.dev), torch.from_numpy(picks.view(np.int32)).to(s.dev),
                            qdelay=torch.from_numpy(qdelay).to(s.dev))
        want = oracle_mod.sub_latency(K, S, w.dag_shared, w.dag_row_ptr, w.dag_col, w.batch, w.workers, w.lat_us, qlen,
                                      gpu.SUB_FULL, lam, samples, picks, threads=8, qdelay=qdelay)
        assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.gpu
@pytest.mark.parametrize("K,n,offset", [(1, 16384, 0), (1, 16385, 0), (4096, 9000, 1), (4097, 9000, 0), (3, 40961, 1), (5, 16, 3), (2, 0, 0), (16385, 16500, 0)])
def test_queue_length_dispatch(gpu, K, n, offset):
    """Both ways of counting at the edges of their rule; offset: the stage array off a 16-byte boundary."""
    import torch
    rng = np.random.default_rng(n + K)
    S = 7
    w = wl.random_workload(5, K=K, S=S, n_per_snapshot=0, dag_shared=1)
    cuts = np.sort(rng.integers(0, n + 1, K - 1))
    snap_ptr = np.concatenate([[0], cuts, [n]]).astype(np.int32)
    stage = rng.integers(-1, S + 1, n).astype(np.int32)
    s = gpu.Session(w)
    d_stage = torch.zeros(n + 4, dtype=torch.int32, device=s.dev)[offset:offset + n]
    d_stage.copy_(torch.from_numpy(stage))
    qlen = torch.full((K * S,), -1, dtype=torch.int32, device=s.dev)
    gpu.pard_queue_lengths(s.plan, n, d_stage, torch.from_numpy(snap_ptr).to(s.dev), qlen)
    torch.cuda.synchronize()
    want = np.concatenate([np.bincount(np.clip(stage[snap_ptr[u]:snap_ptr[u + 1]], 0, S - 1), minlength=S) for u in range(K)])
    assert np.array_equal(qlen.cpu().numpy(), want)
