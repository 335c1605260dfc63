"""The add and drop candidates, collected by chunks of coordinates: vectors at the edges of a chunk, of a workgroup's chunks and of
the workgroups of more threads; rows shifted against each other, crowded chunks, and rows selected from memory."""
import numpy as np
import pytest

from tests.test_gpu_add_drop import GpuAdStepper
from tests.test_gpu_segments import error_buffer_at

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,K,offset,kind", [
    (2, 131_072, 20_000, 1020, "normal"),         # full chunks, two workgroups
    (2, 131_073, 20_000, 4, "normal"),            # ... and three, the last with one coordinate
    (3, 196_608, 20_000, 0, "slow"),              # rows in step with 4 KB; rows selected from memory
    (2, 300_001, 20_000, 8, "crowded"),           # more removals in a workgroup's chunks than are staged at once
    (2, 400_003, 40_000, 512, "turned"),          # nearly all of the standing votes leave
    (2, 98_304, 40_000, 512, "turned"),           # too full for chunks
    (3, 70_001, 700, 4, "normal"),                # short lists
])
def test_candidates_by_chunks(oracle, N, d, K, offset, kind):
    print("[case] ad collect N=%d d=%d K=%d offset=%d %s" % (N, d, K, offset, kind), flush=True)
    rng = np.random.default_rng(d + N)
    gs = GpuAdStepper(N, d, K, K)
    try:
        check_outside = error_buffer_at(gs, offset)
        gs.e[:, :d] = 0
        e, vote, msum = np.zeros((N, d), np.float32), np.zeros((N, d), np.uint8), np.zeros(d, np.uint8)
        for t, k_ad in enumerate([K, max(1, K // 10), K]):
            g = rng.standard_normal((N, d), dtype=np.float32)
            if kind == "crowded":
                g[:, t * 50_000:t * 50_000 + 30_000] *= 100.0
            if kind == "turned":
                g[:, (t & 1) * (d // 2):][:, :d // 2] *= 1000.0 ** (t + 1)
            if kind == "slow":
                g[::2] = 0.5 * (t + 1)
            gs.step(g, k_ad)
            ref = oracle.ad_vote_step(g, e, K, k_ad, vote, msum, threads=8)
            gs.compare(ref, "step %d" % t)
            vote, msum, e = ref.vote, ref.msum, ref.err
        check_outside()
    finally:
        gs.close()
