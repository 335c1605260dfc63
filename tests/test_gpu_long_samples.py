"""The threshold estimate of long rows: on either side of the length from which a row's sample no longer grows, and well beyond it,
the sample finds a list that serves, with and without the samples kept, and the step is the oracle's."""
import numpy as np
import pytest

from paper_2011_06495_amd import binding as B
from tests.gpu_util import GpuStepper, assert_matches_oracle

pytestmark = pytest.mark.gpu

MOST = 131_072 * 128


@pytest.mark.parametrize("N,d,K", [(1, MOST - 33, 8000), (1, MOST + 128, 8000), (2, 24_000_001, 30_000), (5, MOST + 1, 3000),
                                   (2, 40_000_003, 500), (1, 40_000_003, 5000)])       # few: more than a round is sampled
def test_long_rows_are_selected_from_their_lists(oracle, N, d, K):
    print("[case] long samples N=%d d=%d K=%d" % (N, d, K), flush=True)
    rng = np.random.default_rng(d)
    e = np.zeros((N, d), np.float32)
    with GpuStepper(N, d, K) as gs:
        gs.set_error(e)
        for t in range(2):
            g = rng.standard_normal((N, d), dtype=np.float32)
            gs.set_grads(g)
            gs.step()
            ref = oracle.vote_step(g, e, K, threads=8)
            assert_matches_oracle(gs.fetch(), ref, "step %d" % t)
            count, _, slow = B.mv_last_step_row_stats(gs.ctx, N)
            # (seven standard deviations of the sample's count above K, see the rule)
            assert not np.any(np.asarray(slow) == 1) and np.all(np.asarray(count) >= K), (count, slow)
            e = ref.err
