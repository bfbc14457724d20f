"""Large snapshots around the sizes at which a radix pass changes who adds up the digit counts before a tile (16 and 48 chunks of
65,536 requests), with queues few enough for the count kernel to clear the workspace and more than that, on a workspace full of
old values."""
import numpy as np
import pytest

from paper_2602_08747_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8193, 65_537, 16 * 65_536, 16 * 65_536 + 1, 48 * 65_536, 48 * 65_536 + 1])
@pytest.mark.parametrize("queues", [5, 130])
def test_scan_steps(oracle_mod, n, queues):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libpard.so")
    from paper_2602_08747_amd import binding
    if queues == 5:
        w = wl.make_workload(2, n_requests=n, permute=True)
    else:
        K = 26
        w = wl.random_workload(n, K=K, S=5, n_per_snapshot=n // K + 1, time_span=1 << 21, slo_choices=(100_000, 500_000, 900_000),
                               dag_shared=1, vary_sizes=False)
        sizes = np.full(K, n // K)
        sizes[-1] += n - int(sizes.sum())
        w = wl.with_snapshot_sizes(w, np.minimum(sizes, n // K + 1))
    w.lat_us[:] = np.maximum(1, w.lat_us // 300)
    w.now[:] = int(np.median(w.arrival))
    most = max(w.max_snapshot_requests, 8193)
    ref = oracle_mod.run(w, threads=8)
    s = binding.Session(w, max_snapshot_requests=most)
    s.workspace.fill_(0x5A5A5A5A)
    s.workspace[0] = 0
    for _ in range(2):                                    # the second call finds the first one's counts
        s.run()
        got = s.results()
        for k in ("est", "drop", "order", "seg_ptr", "surv_idx", "surv_ptr"):
            assert np.array_equal(got[k], ref[k]), k
    for consistent in (True,) if n < 100_000 else ():
        ref2 = oracle_mod.run(w, threads=8, consistent=True)
        s.workspace.fill_(0x5A5A5A5A)
        s.workspace[0] = 0
        s.run(consistent=consistent)
        got = s.results()
        for k in ("est", "drop", "order", "seg_ptr", "surv_idx", "surv_ptr"):
            assert np.array_equal(got[k], ref2[k]), k
