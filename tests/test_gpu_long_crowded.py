"""Long rows whose magnitudes crowd in the threshold estimate's bin: the threshold is placed inside the bin, and the list stays
near what the sample asks for, although the bin would fit its storage."""
import numpy as np
import pytest

from paper_2011_06495_amd import binding as B
from tests.gpu_util import GpuStepper, assert_matches_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,K,crowd,most", [
    (1, 17_000_003, 17_000, 150_000, 60_000),     # the sample of one round asks for 31,000
    (4, 17_000_000, 30_000, 200_000, 90_000),
    (1, 40_000_003, 500, 52_000, 33_000),         # of several rounds, 16,400
])
def test_crowded_bin_of_a_long_row(oracle, N, d, K, crowd, most):
    print("[case] long crowded N=%d d=%d K=%d crowd=%d" % (N, d, K, crowd), flush=True)
    rng = np.random.default_rng(d)
    g = rng.standard_normal((N, d), dtype=np.float32) * np.float32(0.1)
    for n in range(N):                            # one bin is [1, 1 + 1/32)
        g[n, rng.permutation(d)[:crowd]] = rng.uniform(1.001, 1.03, crowd).astype(np.float32)
    with GpuStepper(N, d, K) as gs:
        e = np.zeros((N, d), np.float32)
        gs.set_error(e)
        gs.set_grads(g)
        gs.step()
        assert_matches_oracle(gs.fetch(), oracle.vote_step(g, e, K, threads=8))
        count, _, slow = B.mv_last_step_row_stats(gs.ctx, N)
        assert not np.any(np.asarray(slow) == 1)
        assert np.all(np.asarray(count) >= K) and np.all(np.asarray(count) <= most), count
