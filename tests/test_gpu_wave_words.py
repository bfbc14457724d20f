"""One wave per snapshot: the 32-bit words and the 64-bit ones on both sides of their rule (bits of stage, key range and index),
and snapshot sizes at the steps of the sorting network."""
import dataclasses

import numpy as np
import pytest

from paper_2602_08747_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("most", [1, 2, 16, 17, 32, 33, 63, 64, 65, 127, 128])
@pytest.mark.parametrize("key_bits", [0, 9, 21, 22, 23, 24, 32])
def test_small_snapshots(oracle_mod, most, key_bits):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libpard.so")
    from paper_2602_08747_amd import binding
    for S, modes in ((4, (wl.MODE_LBF,)), (5, (wl.MODE_HBF,)), (3, (wl.MODE_LBF, wl.MODE_HBF, wl.MODE_FCFS)), (1, (wl.MODE_HBF,))):
        w = wl.random_workload(most + key_bits, K=23, S=S, n_per_snapshot=most, modes=modes, vary_sizes=False)
        rng = np.random.default_rng(most * 40 + key_bits)
        span = (1 << key_bits) - 1
        low = -(1 << 31) if key_bits == 32 else 1000
        d = low + rng.integers(0, span + 1, w.n)
        d[::most], d[most - 1::most] = low, low + span                 # the whole range in every snapshot
        w = dataclasses.replace(w, deadline=d.astype(np.int32), now=np.full_like(w.now, min(low + span // 2, 2**31 - 1)))
        w = wl.with_snapshot_sizes(w, np.where(np.arange(w.K) % 3 == 1, rng.integers(0, most + 1, w.K), most))
        ref = oracle_mod.run(w, threads=4)
        s = binding.Session(w, max_snapshot_requests=most)
        s.run()
        got = s.results()
        for k in ("est", "drop", "order", "seg_ptr", "surv_idx", "surv_ptr"):
            assert np.array_equal(got[k], ref[k]), (k, S, most, key_bits)
