"""The votes of long lists, counted in LDS by chunks of coordinates: vectors at the edges of a chunk, of a workgroup's chunks
and of each chunk length, rows shifted against each other, crowded chunks, and rows selected from memory."""
import numpy as np
import pytest

from paper_2011_06495_amd import binding as B
from tests.gpu_util import GpuStepper, assert_matches_oracle
from tests.test_gpu_segments import error_buffer_at

pytestmark = pytest.mark.gpu


def gradients(rng, N, d, kind):
    if kind == "levels":                          # (quickly drawn)
        return rng.integers(-32768, 32768, (N, d), dtype=np.int16).astype(np.float32)
    g = rng.standard_normal((N, d), dtype=np.float32)
    if kind == "crowded":                         # nearly all votes in a stretch of a few chunks
        g[:, d // 3:d // 3 + 30_000] *= 100.0
    if kind == "slow":                            # equal magnitudes overflow the list: selected from memory
        g[::2] = 0.5
    return g


@pytest.mark.parametrize("N,d,K,offset,kind", [
    (20, (1 << 19) - 1, 27_000, 4, "normal"),     # chunks of 1024
    (20, (1 << 20) - 1, 27_000, 512, "normal"),   # the longest with chunks of 2048, ...
    (5, 1 << 20, 100_000, 0, "normal"),           # ... the shortest with 4096, rows in step with 4 KB
    (5, (1 << 20) + 1, 100_000, 4, "slow"),
    (5, (1 << 20) + 4095, 100_000, 8, "crowded"),
    (13, 4096 * 1024, 40_000, 12, "levels"),      # a chunk to a workgroup, ...
    (13, 4096 * 1024 + 1, 40_000, 1020, "levels"),    # ... and two
    (33, 2_200_003, 20_000, 4, "levels"),
])
@pytest.mark.parametrize("lists", [True, False], ids=["lists", "no_lists"])
def test_votes_by_chunks(oracle, N, d, K, offset, kind, lists):
    print("[case] vote chunks N=%d d=%d K=%d offset=%d %s lists=%s" % (N, d, K, offset, kind, lists), flush=True)
    rng = np.random.default_rng(d + N)
    with GpuStepper(N, d, K, want_worker_idx=lists) as gs:
        check_outside = error_buffer_at(gs, offset)
        e = np.zeros((N, d), np.float32)
        gs.set_error(e)
        for t in range(1 if kind == "levels" else 2):
            g = gradients(rng, N, d, kind)
            gs.set_grads(g)
            B.mv_set_profiling(gs.ctx, 2)
            gs.step()
            ms = dict(zip(B.kernel_names(), B.mv_step_kernel_ms(gs.ctx)))
            assert ms["mv_vote_count"] >= 0
            ref = oracle.vote_step(g, e, K, threads=8)
            assert_matches_oracle(gs.fetch(), ref, "step %d" % t)
            e = ref.err
        check_outside()
