"""Lists that many workgroups select from (large K): the rows' candidates, the add and drop candidates and the random
selection, against the oracle.  Values that spread the boundary over one bin, over thousands of members of one bin
(beyond what is ranked in on-chip memory), over equal magnitudes, and rows that have to be selected from memory."""
import sys

import numpy as np
import pytest
import torch

from paper_2011_06495_amd import binding as B
from tests.gpu_util import GpuStepper, assert_matches_oracle
from tests.test_gpu_add_drop import GpuAdStepper

pytestmark = pytest.mark.gpu


def values(rng, kind, N, d):
    g = rng.standard_normal((N, d))
    if kind == "lattice":            # about a hundred magnitudes
        g = np.round(g * 24.0) / 64.0
    elif kind == "crowded":          # the largest 40 % within 2^-11 of each other
        g = np.where(rng.random((N, d)) < 0.4, 1.0 + rng.random((N, d)) * 2.0 ** -11, g * 1e-3)
    elif kind == "far":              # the boundary lies octaves above the estimate for some, ties for others
        g = np.where(rng.random((N, d)) < 0.12, 8.0 + rng.random((N, d)) * 40.0, np.round(g * 3) / 4)
    elif kind == "degenerate":       # one magnitude, zeros, and an ordinary row
        g[0] = 2.5
        g[1] = 0.0
    return g.astype(np.float32)


@pytest.mark.parametrize("kind", ["normal", "lattice", "crowded", "far", "degenerate"])
@pytest.mark.parametrize("N,d,K", [(3, 300007, 30000), (4, 131075, 26001)])
def test_rows_and_random_selection(oracle, kind, N, d, K):
    print("[case] long lists %s N=%d d=%d K=%d" % (kind, N, d, K), flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(sum(map(ord, kind)) + d)
    e = np.zeros((N, d), np.float32)
    clocks = [np.ones(d), rng.integers(1, 4, d), 1.0 + rng.random(d) * 2.0 ** -12, rng.standard_exponential(d)]
    with GpuStepper(N, d, K) as gs:
        gs.set_error(e)
        for t in range(6):
            g = values(rng, kind, N, d)
            gs.set_grads(g)
            if t == 1:
                B.mv_set_spin_limit(gs.ctx, 0)        # rows whose threshold is not seen at once go the exact way
            if t == 2:
                B.mv_set_spin_limit(gs.ctx, 1 << 20)
            if t < 2:
                gs.step()
                ref = oracle.vote_step(g, e, K, threads=8)
            else:
                r = clocks[t - 2].astype(np.float32)
                gs.step_rs(r)
                ref = oracle.rs_vote_step(g, e, K, r, threads=8)
            assert_matches_oracle(gs.fetch(), ref, "%s step %d" % (kind, t))
            e = ref.err


@pytest.mark.parametrize("kind", ["normal", "lattice", "crowded", "degenerate"])
@pytest.mark.parametrize("N,d,K", [(3, 300007, 30000), (2, 90001, 16384), (2, 90001, 16385)])
def test_additions_and_removals(oracle, kind, N, d, K):
    print("[case] long add-drop lists %s N=%d d=%d K=%d" % (kind, N, d, K), flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(sum(map(ord, kind)) + K)
    gs = GpuAdStepper(N, d, K, K)
    try:
        vote, msum, e = np.zeros((N, d), np.uint8), np.zeros(d, np.uint8), np.zeros((N, d), np.float32)
        for t, k_ad in enumerate([K, K // 4, 1, 9000, K]):
            g = values(rng, kind, N, d)
            ref = oracle.ad_vote_step(g, e, K, k_ad, vote, msum, threads=8)
            gs.step(g, k_ad)
            gs.compare(ref, "%s step %d k_ad %d" % (kind, t, k_ad))
            vote, msum, e = ref.vote, ref.msum, ref.err
    finally:
        gs.close()


@pytest.mark.parametrize("N,K,votes", [(2, 4096, "shared"), (1, 16384, "own"), (4, 4097, "own"), (5, 3277, "own")])
def test_random_selection_around_one_workgroups_list(oracle, N, K, votes):
    """Lists of 4096 to 16,385 voted coordinates: a batch of one workgroup, all that one workgroup takes, one more."""
    d = 70001
    print("[case] random selection N=%d K=%d votes %s" % (N, K, votes), flush=True)
    rng = np.random.default_rng(N * K)
    g = np.full((N, d), 1e-3, np.float32)
    for n in range(N):
        at = np.arange(K) if votes == "shared" else np.arange(n * K, (n + 1) * K)
        g[n, at % d] = 1.0 + rng.random(K)
    e = np.zeros_like(g)
    for r in (rng.standard_exponential(d).astype(np.float32), np.full(d, 0.5, np.float32)):
        with GpuStepper(N, d, K) as gs:
            gs.set_error(e)
            gs.set_grads(g)
            gs.step_rs(r)
            assert_matches_oracle(gs.fetch(), oracle.rs_vote_step(g, e, K, r), "N=%d K=%d" % (N, K))


@pytest.mark.parametrize("m", [3071, 3072, 3073, 8191, 8192, 8193])
def test_groups_around_what_fits_on_chip(oracle, m):
    """The boundary lies in a group of m equal magnitudes (m equal times): 3072 members of a bin are kept in LDS in the
    rows' select and for the add and drop lists, 8192 in the random selection."""
    N, d, K = 2, 300007, 32000
    print("[case] groups around what fits on chip m=%d" % m, flush=True)
    rng = np.random.default_rng(m)
    above = K - m // 2
    g = rng.uniform(0.1, 0.9, (N, d)).astype(np.float32)
    for n in range(N):
        at = rng.permutation(d)
        g[n, at[:above]] = rng.uniform(2.0, 3.0, above)
        g[n, at[above:above + m]] = 1.0
    e = np.zeros_like(g)
    with GpuStepper(N, d, K) as gs:
        gs.set_grads(g)
        gs.set_error(e)
        gs.step()
        ref = oracle.vote_step(g, e, K, threads=8)
        assert_matches_oracle(gs.fetch(), ref, "plain")
        once = rng.permutation(np.flatnonzero(ref.votes == 1))
        r = np.full(d, 3.0, np.float32)
        r[once[:above]] = rng.uniform(0.1, 0.4, above)
        r[once[above:above + m]] = 1.0
        gs.set_grads(g)
        gs.set_error(e)
        gs.step_rs(r)
        assert_matches_oracle(gs.fetch(), oracle.rs_vote_step(g, e, K, r, threads=8), "random")
