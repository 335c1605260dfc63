"""The votes of crowded chunks: long runs of list entries are walked by a wavefront each, short ones dealt to the threads entry by
entry, and the pieces of very crowded chunks dealt round the grid.  Runs around the length from which they are long and around a wavefront's loads, whole segments, chunks of each length,
rows that begin anywhere, crowded coordinates at the vector's end and elsewhere in the next step, and rows from memory beside."""
import numpy as np
import pytest

from paper_2011_06495_amd import binding as B
from tests.gpu_util import GpuStepper, assert_matches_oracle
from tests.test_gpu_segments import error_buffer_at

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,K,offset,hot,gain,slow", [
    (5, 1 << 20, 100_000, 0, 20_000, 100, False),         # chunks of 4096, rows in step with 4 KB
    (5, (1 << 20) + 4095, 100_000, 8, 9_000, 100, False),
    (20, (1 << 20) - 1, 27_000, 1020, 20_000, 100, True),     # of 2048; every other row from memory
    (20, (1 << 19) - 1, 27_000, 4, 20_000, 100, False),   # of 1024
    (8, 4_200_001, 100_000, 512, 130_000, 100, False),    # runs of whole segments, two chunks to a workgroup
    (8, 4_200_001, 100_000, 4, 500_000, 100, False),      # of about 256 entries
    (8, 4_200_001, 100_000, 1020, 1_000_000, 100, False),     # of about 128
])
@pytest.mark.parametrize("lists", [True, False], ids=["lists", "no_lists"])
def test_crowded_chunks(oracle, N, d, K, offset, hot, gain, slow, lists):
    crowded_steps(oracle, N, d, K, offset, hot, gain, slow, lists, 2)


def test_more_pieces_than_workgroups(oracle):
    """257 very crowded chunks of 4096 for 1023 workgroups."""
    crowded_steps(oracle, 64, 4_190_001, 21_000, 4, 1_050_000, 100, False, True, 1)


def test_more_rows_than_are_counted_in_chunks_of_4096(oracle):
    """Chunks of 2048 in a vector of millions."""
    crowded_steps(oracle, 205, 6_000_001, 15_000, 1020, 600_000, 2, False, True, 1)


def crowded_steps(oracle, N, d, K, offset, hot, gain, slow, lists, steps):
    print("[case] crowded N=%d d=%d K=%d offset=%d hot=%d lists=%s" % (N, d, K, offset, hot, lists), flush=True)
    rng = np.random.default_rng(d + N)
    with GpuStepper(N, d, K, want_worker_idx=lists) as gs:
        check_outside = error_buffer_at(gs, offset)
        e = np.zeros((N, d), np.float32)
        gs.set_error(e)
        B.mv_set_profiling(gs.ctx, 2)
        for t in range(steps):
            print("[case] step %d" % t, flush=True)
            g = rng.integers(-32768, 32768, (N, d), dtype=np.int16).astype(np.float32)
            start = d - hot if t == 0 else d // 3         # up to the end, then elsewhere
            g[:, start:start + hot] *= gain
            if slow:
                g[::2] = 0.5 * (t + 1)
            gs.set_grads(g)
            gs.step()
            ms = dict(zip(B.kernel_names(), B.mv_step_kernel_ms(gs.ctx)))
            assert ms["mv_vote_count"] >= 0
            from_memory = np.asarray(gs.row_stats()[2]) == 1
            assert np.array_equal(from_memory, (np.arange(N) % 2 == 0) & slow), from_memory
            ref = oracle.vote_step(g, e, K, threads=8)
            assert_matches_oracle(gs.fetch(), ref, "step %d" % t)
            e = ref.err
        check_outside()
