"""The add and drop candidates of long, dense lists come from the kernel that goes by chunks of coordinates, the others from the
one that looks candidates up, each timed under its own name: vectors at the edges of a workgroup's chunks, rows shifted against
each other, more removals than are staged at once, and rows selected from memory."""
import numpy as np
import pytest

from paper_2011_06495_amd import binding as B
from tests.test_gpu_add_drop import GpuAdStepper
from tests.test_gpu_segments import error_buffer_at

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,K,offset,kind,chunks", [
    (2, 262_144, 27_000, 0, "normal", True),      # four workgroups of full chunks, rows in step with 4 KB
    (2, 262_145, 27_000, 4, "normal", True),      # ... and a fifth with one coordinate
    (3, 327_680, 27_000, 1020, "normal", True),
    (3, 1_000_003, 40_000, 8, "slow", True),      # equal magnitudes overflow the list: selected from memory
    (2, 300_001, 25_000, 512, "crowded", True),   # more removals in a workgroup's chunks than are staged at once
    (3, 400_003, 40_000, 4, "turned", True),      # nearly all of the standing votes leave
    (2, 262_145, 70_000, 1020, "normal", True),   # full lists
    (3, 400_003, 80_000, 4, "crowded", True),
    (2, 786_432, 200_000, 0, "turned", True),
    (2, 131_073, 20_000, 4, "normal", False),     # lists that one workgroup selects
    (2, 98_304, 40_000, 512, "normal", False),    # too full for chunks
])
def test_collecting_kernel(oracle, N, d, K, offset, kind, chunks):
    print("[case] ad collect route N=%d d=%d K=%d offset=%d %s" % (N, d, K, offset, kind), flush=True)
    rng = np.random.default_rng(d + N)
    gs = GpuAdStepper(N, d, K, K)
    try:
        check_outside = error_buffer_at(gs, offset)
        gs.e[:, :d] = 0
        B.mv_set_profiling(gs.ctx, 2)
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
            ms = dict(zip(B.kernel_names(), B.mv_step_kernel_ms(gs.ctx)))
            assert (ms["mv_ad_collect_chunks"] >= 0) == chunks and (ms["mv_ad_collect"] >= 0) == (not chunks)
            from_memory = np.asarray(B.mv_last_step_row_stats(gs.ctx, N)[2]) == 1
            assert np.array_equal(from_memory, (np.arange(N) % 2 == 0) & (kind == "slow")), from_memory
            ref = oracle.ad_vote_step(g, e, K, k_ad, vote, msum, threads=8)
            gs.compare(ref, "step %d" % t)
            vote, msum, e = ref.vote, ref.msum, ref.err
        check_outside()
    finally:
        gs.close()
