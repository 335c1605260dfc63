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


def tied_values(rng, kind, N, d):
    if kind == "equal":              # one magnitude: the candidate list is the row, with no room behind it
        g = np.where(rng.random((N, d)) < 0.5, -2.5, 2.5)
    elif kind == "lattice":
        g = np.round(rng.standard_normal((N, d)) * 6.0) / 64.0
    elif kind == "zeros":            # the boundary lies among zeros
        g = np.where(rng.random((N, d)) < 0.05, rng.standard_normal((N, d)), 0.0)
    elif kind == "one_bin":          # thousands of different keys within one bin, many of them several times
        g = 1.0 + rng.integers(0, 3000, (N, d)) * 2.0 ** -23
    else:                            # "two_bins": a tie group in a wide bin far above the estimate's, beside another key
        g = np.where(rng.random((N, d)) < 0.3, 8.0 + np.round(rng.random((N, d))) * 2.0 ** -8,
                     rng.standard_normal((N, d)) * 1e-2)
    return g.astype(np.float32)


@pytest.mark.parametrize("kind", ["equal", "lattice", "zeros", "one_bin", "two_bins"])
@pytest.mark.parametrize("N,d,K", [(3, 200003, 40000), (3, 200003, 150002), (2, 200003, 200002), (2, 200003, 200003),
                                   (2, 60001, 57000), (2, 2500003, 500000), (2, 2097153, 1900000)])
def test_large_tie_groups(oracle, kind, N, d, K):
    """Tie groups far larger than what is ranked in on-chip memory, with room for them behind the list and without, in
    rows whose blocks of coordinates have one segment and two; several steps of one context."""
    print("[case] large tie groups %s N=%d d=%d K=%d" % (kind, N, d, K), flush=True)
    rng = np.random.default_rng(sum(map(ord, kind)) + K)
    e = np.zeros((N, d), np.float32)
    with GpuStepper(N, d, K) as gs:
        gs.set_error(e)
        for t in range(3):
            g = tied_values(rng, kind, N, d)
            gs.set_grads(g)
            if t != 1:
                gs.step()
                ref = oracle.vote_step(g, e, K, threads=8)
            else:
                r = rng.standard_exponential(d).astype(np.float32)
                gs.step_rs(r)
                ref = oracle.rs_vote_step(g, e, K, r, threads=8)
            assert_matches_oracle(gs.fetch(), ref, "%s step %d" % (kind, t))
            e = ref.err
    gs = GpuAdStepper(N, d, K, K)
    try:
        vote, msum, e = np.zeros((N, d), np.uint8), np.zeros(d, np.uint8), np.zeros((N, d), np.float32)
        for t, k_ad in enumerate([K, K // 3, 100]):
            g = tied_values(rng, kind, N, d)
            ref = oracle.ad_vote_step(g, e, K, k_ad, vote, msum, threads=8)
            gs.step(g, k_ad)
            gs.compare(ref, "%s add-drop step %d k_ad %d" % (kind, t, k_ad))
            vote, msum, e = ref.vote, ref.msum, ref.err
    finally:
        gs.close()


def test_large_tie_groups_are_not_left_to_one_workgroup():
    """A row of equal magnitudes costs about what an ordinary row does: its tie group is neither ranked nor voted for
    by one workgroup member by member (which took 50 times as long)."""
    N, d, K = 2, 1000003, 500001
    print("[case] time of large tie groups N=%d d=%d K=%d" % (N, d, K), flush=True)

    def milliseconds(kind):
        best = 1e9
        with GpuStepper(N, d, K) as gs:
            gs.set_grads(np.random.default_rng(1).standard_normal((N, d)) if kind == "normal" else np.full((N, d), 2.5))
            for _ in range(6):
                gs.set_error(np.zeros((N, d), np.float32))
                start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                start.record()
                gs.step()
                end.record()
                torch.cuda.synchronize()
                best = min(best, start.elapsed_time(end))
        return best

    ordinary, equal = milliseconds("normal"), milliseconds("equal")
    print("  ordinary %.3f ms, equal %.3f ms" % (ordinary, equal), flush=True)
    assert equal < 8 * ordinary


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


@pytest.mark.parametrize("N,d,K", [(2, 300007, 40000), (1, 150001, 30000), (3, 90001, 41000)])
@pytest.mark.parametrize("magnitudes", ["equal", "one_bin", "spread"])
def test_lists_of_exactly_k(oracle, N, d, K, magnitudes):
    """Rows with exactly K coordinates that are not zero, elsewhere in every step: the list is the vote, and what left
    it -- zeros now -- is outside the top K.  (All workers have the same support, so every step transmits all of it.)"""
    print("[case] lists of exactly K %s N=%d d=%d K=%d" % (magnitudes, N, d, K), flush=True)
    rng = np.random.default_rng(K + len(magnitudes))
    gs = GpuAdStepper(N, d, K, K)
    try:
        vote, msum, e = np.zeros((N, d), np.uint8), np.zeros(d, np.uint8), np.zeros((N, d), np.float32)
        for t, k_ad in enumerate([K, K, K // 2, K]):
            g = np.zeros((N, d), np.float32)
            at = rng.permutation(d)[:K]
            v = {"equal": np.ones((N, K)), "one_bin": 1.0 + rng.integers(0, 4000, (N, K)) * 2.0 ** -23,
                 "spread": 1.0 + rng.random((N, K))}[magnitudes]
            g[:, at] = v
            ref = oracle.ad_vote_step(g, e, K, k_ad, vote, msum, threads=8)
            gs.step(g, k_ad)
            gs.compare(ref, "step %d" % t)
            vote, msum, e = ref.vote, ref.msum, ref.err
    finally:
        gs.close()


@pytest.mark.parametrize("kind,N,d,K", [("lattice", 128, 200_003, 20_000), ("normal", 255, 70_001, 12_000)])
def test_sorted_lists_without_room_beside_the_vote_blocks(oracle, kind, N, d, K):
    """More than 512 workgroups with the vote blocks' (one quad per thread): the lists are written beside the gather."""
    print("[case] lists beside the gather %s N=%d d=%d K=%d" % (kind, N, d, K), flush=True)
    rng = np.random.default_rng(N + d)
    g = values(rng, kind, N, d)
    g[1] = 0.0                                        # a row selected from memory, whose list is written by then
    e = np.zeros((N, d), np.float32)
    with GpuStepper(N, d, K) as gs:
        for t in range(2):
            gs.set_error(e)
            gs.set_grads(g)
            gs.step()
            assert_matches_oracle(gs.fetch(), oracle.vote_step(g, e, K, threads=8), "%s step %d" % (kind, t))
