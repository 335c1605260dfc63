"""The mask kernel's stretches: lengths at and around the edges of a wavefront's kilobytes of votes and of a block, for
one to four quads per thread, with the blocks' exchange and (nobody waiting) with the gather finding the mask."""
import numpy as np
import pytest

from paper_2011_06495_amd import binding as B
from tests.gpu_util import GpuStepper, assert_matches_oracle

pytestmark = pytest.mark.gpu

BLOCK = 16384                                     # vote bytes of a block with one quad per thread


def most(N, quads):
    """The longest vector whose blocks have so many quads per thread."""
    return (500 - N) * BLOCK * quads


@pytest.mark.parametrize("N,d", [(3, 2 * BLOCK + 1), (3, 2 * BLOCK + 1023), (3, 2 * BLOCK + 1024), (2, 3 * BLOCK), (2, 5 * BLOCK + 1039),
                                 (2, most(2, 1)), (2, most(2, 1) + 1), (2, most(2, 1) + 2048 + 15), (1, most(1, 2) + 1024),
                                 (1, most(1, 3) + 17)])
@pytest.mark.parametrize("wait", [True, False], ids=["exchange", "gather_finds"])
def test_votes_and_mask_at_the_edges_of_stretches(oracle, N, d, wait):
    print("[case] stretches N=%d d=%d wait=%s" % (N, d, wait), flush=True)
    K = max(64, d // 1500)
    rng = np.random.default_rng(d)
    g = np.rint(rng.standard_normal((N, d), dtype=np.float32) * 8.0) / 8.0       # ties at every threshold
    g[:, -3:] = 100.0                             # the last coordinates are in every vote
    e = np.zeros((N, d), np.float32)
    ref = oracle.vote_step(g, e, K, threads=8)
    with GpuStepper(N, d, K) as gs:
        if not wait:
            B.mv_set_spin_limit(gs.ctx, 0)
        gs.set_error(e)
        gs.set_grads(g)
        gs.step()
        assert_matches_oracle(gs.fetch(), ref, "N=%d d=%d" % (N, d))
