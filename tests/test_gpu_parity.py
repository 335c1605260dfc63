"""Parity of the HIP path (through the C ABI) against the CPU oracle, element by
element on the same seeded inputs.  Index sets, votes, mask and the error
buffer must be bit-exact; the aggregate within 1e-6 relative (it is bit-exact,
the worker order of the sum being fixed on both sides)."""
import sys

import numpy as np
import pytest
import torch

from paper_2011_06495_amd import binding as B
from paper_2011_06495_amd import workloads as W
from tests.gpu_util import GpuStepper, assert_matches_oracle
from tests.test_gpu_add_drop import GpuAdStepper

pytestmark = pytest.mark.gpu


def say(msg):
    print("[case] " + msg, flush=True)
    sys.stdout.flush()


def run_sequence(oracle, w, steps, e0=None, threads=8, **kw):
    """Runs `steps` consecutive vote steps on both sides with the error buffer
    carried, comparing after every step."""
    e_ref = W.zero_error(w) if e0 is None else e0.copy()
    with GpuStepper(w.N, w.d, w.K, bf16=(w.grad_dtype == "bf16"), **kw) as gs:
        gs.set_error(e_ref)
        for t in range(steps):
            g = W.gradients(w, t)
            gs.set_grads(g)
            gs.step()
            got = gs.fetch()
            ref = oracle.vote_step(g, e_ref, w.K, threads=threads)
            assert_matches_oracle(got, ref, "%s step %d" % (w.name, t))
            e_ref = ref.err
        return gs.row_stats()


# several tiles of every kernel and a ragged tail: d is not a multiple of 4, 16, 32, 1024 or 16384
SMALL = {
    "C1": W.C1.with_size(150001),
    "C2": W.C2.with_size(300007, N=10),
    "C3": W.C3.with_size(257003, N=16),
    "C4": W.C4.with_size(200003, N=16, lattice_shift=6),
    "C5": W.C5.with_size(180005, N=32),
}


@pytest.mark.parametrize("name", sorted(SMALL))
def test_reduced_workloads_three_steps(oracle, name):
    w = SMALL[name]
    say("reduced %s N=%d d=%d K=%d" % (name, w.N, w.d, w.K))
    run_sequence(oracle, w, 3)


@pytest.mark.parametrize("d,K,N", [(1, 1, 1), (2, 1, 3), (5, 5, 2), (31, 7, 4), (1023, 10, 3), (1024, 1024, 2),
                                   (1025, 3, 5), (4097, 1, 2), (16385, 100, 3), (70001, 69999, 2),
                                   (50000, 500, 255)])
def test_edge_shapes(oracle, d, K, N):
    say("edge shape d=%d K=%d N=%d" % (d, K, N))
    rng = np.random.default_rng(d * 7 + K)
    g = rng.standard_normal((N, d)).astype(np.float32)
    e = (rng.standard_normal((N, d)) * 0.1).astype(np.float32)
    with GpuStepper(N, d, K) as gs:
        gs.set_error(e)
        gs.set_grads(g)
        gs.step()
        assert_matches_oracle(gs.fetch(), oracle.vote_step(g, e, K), "d=%d K=%d N=%d" % (d, K, N))


def test_degenerate_rows_take_the_exact_slow_path(oracle):
    """All-zero, all-equal and two-valued rows: the estimate cannot separate K
    coordinates, the row is selected exactly from memory, lowest index first."""
    N, d, K = 5, 140003, 137
    say("degenerate rows N=%d d=%d K=%d" % (N, d, K))
    rng = np.random.default_rng(1)
    g = np.zeros((N, d), np.float32)
    g[1] = -2.5
    g[2] = rng.choice(np.array([1.0, -1.0, 3.0], np.float32), size=d)      # huge tie groups
    g[3] = rng.standard_normal(d).astype(np.float32)
    g[4, ::2] = -0.0
    e = np.zeros_like(g)
    with GpuStepper(N, d, K) as gs:
        gs.set_error(e)
        gs.set_grads(g)
        gs.step()
        got = gs.fetch()
        _, _, slow = gs.row_stats()
    ref = oracle.vote_step(g, e, K)
    assert_matches_oracle(got, ref, "degenerate")
    assert got.worker_idx[0].tolist() == list(range(K))
    assert got.worker_idx[1].tolist() == list(range(K))
    assert slow[0] == 1 and slow[1] == 1 and slow[3] != 1


def test_denormals_and_signed_zero_are_ordered_not_flushed(oracle):
    N, d, K = 2, 5000, 40
    say("denormals N=%d d=%d K=%d" % (N, d, K))
    rng = np.random.default_rng(2)
    bits = rng.integers(1, 1 << 20, size=(N, d)).astype(np.uint32)          # denormal magnitudes
    bits |= (rng.integers(0, 2, size=(N, d)).astype(np.uint32) << 31)
    g = bits.view(np.float32)
    e = np.zeros_like(g)
    e[:, ::3] = g[:, ::3]                                                   # denormal + denormal
    with GpuStepper(N, d, K) as gs:
        gs.set_error(e)
        gs.set_grads(g)
        gs.step()
        got = gs.fetch()
    ref = oracle.vote_step(g, e, K)
    assert np.count_nonzero(ref.err) > 0
    assert_matches_oracle(got, ref, "denormals")


def test_row_stride_larger_than_d_and_padding_untouched(oracle):
    w = W.C2.with_size(33331, N=3)
    say("strided rows d=%d" % w.d)
    run_sequence(oracle, w, 2, extra_ld=5)


@pytest.mark.parametrize("w", [W.C2.with_size(40001, N=7), W.C2.with_size(20011, N=255), W.C5.with_size(60005, N=5)],
                         ids=["f32_N7", "f32_N255", "bf16_N5"])
def test_sum_reduction(oracle, w):
    say("sum reduction N=%d d=%d K=%d %s" % (w.N, w.d, w.K, w.grad_dtype))
    e = W.zero_error(w)
    with GpuStepper(w.N, w.d, w.K, bf16=(w.grad_dtype == "bf16"), reduce=B.MV_REDUCE_SUM) as gs:
        gs.set_error(e)
        for t in range(2):                                                 # the second step with a carried error
            g = W.gradients(w, t)
            gs.set_grads(g)
            gs.step()
            got = gs.fetch()
            ref = oracle.vote_step(g, e, w.K, reduce_mean=False)
            assert_matches_oracle(got, ref, "sum, step %d" % t)
            e = ref.err


def test_infinite_magnitudes_are_ordered_above_finite(oracle):
    """+-Inf is a magnitude like any other, above every finite one; equal infinities go to the
    lowest coordinate.  (Coordinates where Inf - Inf would arise are outside the contract and
    not produced here: at a coordinate the infinities of all workers have one sign.)"""
    N, d, K = 3, 70001, 500
    say("infinities N=%d d=%d K=%d" % (N, d, K))
    rng = np.random.default_rng(11)
    g0 = rng.standard_normal((N, d)).astype(np.float32)
    sign = np.where(rng.integers(0, 2, size=d) == 1, np.float32(np.inf), np.float32(-np.inf))
    few = rng.choice(d, size=40, replace=False)
    g0[0, few] = sign[few]
    g0[2, few[:25]] = sign[few[:25]]
    many = rng.choice(d, size=K + 100, replace=False)                      # more infinities than K: ties among them
    g0[1, many] = sign[many]
    g1 = rng.standard_normal((N, d)).astype(np.float32)                    # finite: Inf + finite stays Inf
    e = np.zeros((N, d), np.float32)
    with GpuStepper(N, d, K) as gs:
        gs.set_error(e)
        for t, g in enumerate((g0, g1)):
            gs.set_grads(g)
            gs.step()
            got = gs.fetch()
            ref = oracle.vote_step(g, e, K)
            assert not np.isnan(ref.agg).any() and not np.isnan(ref.err).any()
            assert np.isinf(ref.agg).any()
            assert_matches_oracle(got, ref, "infinities, step %d" % t)
            e = ref.err
        assert np.isinf(e).any()                                           # infinities that lost the vote were carried


def test_nan_inputs_end_with_valid_indices():
    """NaN is outside the contract (its payload after an addition is the processor's choice): the
    values are then unspecified, but the step ends and every index it writes is a coordinate."""
    N, d, K = 4, 50003, 300
    say("NaN N=%d d=%d K=%d" % (N, d, K))
    rng = np.random.default_rng(12)
    g = rng.standard_normal((N, d)).astype(np.float32)
    g[rng.integers(0, N, size=2000), rng.integers(0, d, size=2000)] = np.float32(np.nan)
    g[1, :400] = np.float32(np.inf)
    e = np.zeros((N, d), np.float32)
    e[1, :200] = np.float32(-np.inf)                                       # Inf - Inf
    with GpuStepper(N, d, K) as gs:
        gs.set_error(e)
        gs.set_grads(g)
        gs.step()
        got = gs.fetch()
    assert np.all(got.mask_idx < d) and np.all(np.diff(got.mask_idx.astype(np.int64)) > 0)
    assert np.all(got.worker_idx < d) and np.all(np.diff(got.worker_idx.astype(np.int64), axis=1) > 0)
    assert got.votes.max() <= N and int(got.votes.sum()) == N * K
    assert np.all(got.err[:, got.mask_idx].view(np.uint32) == 0)


def test_mask_is_exact_when_the_blocks_do_not_wait_for_each_other(oracle):
    """With no polls allowed, a streaming wavefront that does not find its row's threshold at the
    first look gives the row to the exact slow path, and a block of the mask kernel that does not
    find the earlier blocks' counts at the first look leaves the mask to the kernel behind it:
    slower, and the same result."""
    w = W.C4.with_size(700001, N=6)
    say("no polls N=%d d=%d K=%d" % (w.N, w.d, w.K))
    e = W.zero_error(w)
    with GpuStepper(w.N, w.d, w.K) as gs:
        B.mv_set_spin_limit(gs.ctx, 0)
        gs.set_error(e)
        for t in range(2):
            g = W.gradients(w, t)
            gs.set_grads(g)
            gs.step()
            got = gs.fetch()
            ref = oracle.vote_step(g, e, w.K)
            assert_matches_oracle(got, ref, "no polls, step %d" % t)
            e = ref.err


def test_optional_outputs_and_caller_workspace(oracle):
    w = W.C3.with_size(90001, N=6)
    say("optional outputs / caller workspace")
    g, e = W.gradients(w, 0), W.zero_error(w)
    ref = oracle.vote_step(g, e, w.K)
    for kw in (dict(want_worker_idx=False), dict(want_votes=False), dict(own_workspace=True),
               dict(want_worker_idx=False, want_votes=False, own_workspace=True)):
        with GpuStepper(w.N, w.d, w.K, **kw) as gs:
            gs.set_error(e)
            gs.set_grads(g)
            gs.step()
            assert_matches_oracle(gs.fetch(), ref, str(kw))


def test_result_does_not_depend_on_context_history(oracle):
    """A context that has run other data gives the same bits as a fresh one, and
    the same call twice gives the same bits (atomics only order scratch)."""
    w = W.C4.with_size(120001, N=8, lattice_shift=6)
    say("determinism / history independence")
    g0, g1 = W.gradients(w, 0), W.gradients(w, 1)
    e = W.zero_error(w)
    outs = []
    with GpuStepper(w.N, w.d, w.K) as gs:
        for g in (g0, g1, g0):
            gs.set_error(e)
            gs.set_grads(g)
            gs.step()
            outs.append(gs.fetch())
    with GpuStepper(w.N, w.d, w.K) as gs:
        gs.set_error(e)
        gs.set_grads(g0)
        gs.step()
        fresh = gs.fetch()
    for other in (outs[2], fresh):
        assert np.array_equal(outs[0].worker_idx, other.worker_idx)
        assert np.array_equal(outs[0].votes, other.votes)
        assert np.array_equal(outs[0].mask_idx, other.mask_idx)
        assert np.array_equal(outs[0].agg.view(np.uint32), other.agg.view(np.uint32))
        assert np.array_equal(outs[0].err.view(np.uint32), other.err.view(np.uint32))
    assert_matches_oracle(outs[0], oracle.vote_step(g0, e, w.K), "history")


def test_resume_through_host_copy_of_error_buffer(oracle):
    """The error buffer is the only state: 6 steps == 3 steps, E to host and into
    a new context, 3 more steps."""
    w = W.C3.with_size(60001, N=4, steps=6)
    say("resume")
    with GpuStepper(w.N, w.d, w.K) as gs:
        gs.set_error(W.zero_error(w))
        for t in range(6):
            gs.set_grads(W.gradients(w, t))
            gs.step()
        full = gs.fetch()
    with GpuStepper(w.N, w.d, w.K) as gs:
        gs.set_error(W.zero_error(w))
        for t in range(3):
            gs.set_grads(W.gradients(w, t))
            gs.step()
        half = gs.fetch()
    with GpuStepper(w.N, w.d, w.K) as gs:
        gs.set_error(half.err)
        for t in range(3, 6):
            gs.set_grads(W.gradients(w, t))
            gs.step()
        resumed = gs.fetch()
    assert np.array_equal(full.mask_idx, resumed.mask_idx)
    assert np.array_equal(full.err.view(np.uint32), resumed.err.view(np.uint32))
    assert np.array_equal(full.agg.view(np.uint32), resumed.agg.view(np.uint32))


def test_non_default_stream(oracle):
    w = W.C2.with_size(50001, N=4)
    say("side stream")
    g, e = W.gradients(w, 0), W.zero_error(w)
    s = torch.cuda.Stream()
    with GpuStepper(w.N, w.d, w.K) as gs:
        gs.set_error(e)
        gs.set_grads(g)
        torch.cuda.synchronize()
        gs.step(stream=s)
        s.synchronize()
        assert_matches_oracle(gs.fetch(), oracle.vote_step(g, e, w.K), "stream")


def test_argument_errors_leave_error_buffer_untouched():
    say("argument errors on a live context")
    with GpuStepper(2, 1000, 10) as gs:
        gs.set_error(np.ones((2, 1000), np.float32))
        L = B.load()
        st = L.mv_vote_step(gs.ctx, gs.g.data_ptr(), 999, gs.e.data_ptr(), gs.ld_e, 0, 0,
                            gs.mask.data_ptr(), gs.agg.data_ptr(), 0)
        assert st == B.MV_ERR_INVALID_ARG                       # ld < d
        st = L.mv_vote_step(gs.ctx, gs.g.data_ptr() + 4, gs.ld_g, gs.e.data_ptr(), gs.ld_e, 0, 0,
                            gs.mask.data_ptr(), gs.agg.data_ptr(), 0)
        assert st == B.MV_ERR_INVALID_ARG                       # misaligned
        st = L.mv_vote_step(gs.ctx, gs.g.data_ptr(), gs.ld_g, gs.e.data_ptr(), gs.ld_e, 0, 0,
                            0, gs.agg.data_ptr(), 0)
        assert st == B.MV_ERR_INVALID_ARG                       # null mask
        torch.cuda.synchronize()
        assert torch.all(gs.e[:, :1000] == 1.0)
        ctx = gs.ctx
        B.mv_end(ctx)
        st = L.mv_vote_step(ctx, gs.g.data_ptr(), gs.ld_g, gs.e.data_ptr(), gs.ld_e, 0, 0,
                            gs.mask.data_ptr(), gs.agg.data_ptr(), 0)
        assert st == B.MV_ERR_STATE
        assert L.mv_end(ctx) == B.MV_ERR_STATE
        B.mv_release(ctx)
        gs.ctx = 0


def _levels_row(rng, d, groups, noise=1e-3):
    """A row of small noise with groups of (count, lo, hi) magnitudes planted at random places."""
    row = (rng.standard_normal(d) * noise).astype(np.float32)
    pos = rng.permutation(d)
    at = 0
    for count, lo, hi in groups:
        vals = rng.uniform(lo, hi, size=count).astype(np.float32) if hi > lo else np.full(count, lo, np.float32)
        row[pos[at:at + count]] = vals * rng.choice(np.array([-1.0, 1.0], np.float32), size=count)
        at += count
    return row


@pytest.mark.parametrize("case", ["ties_in_lds_by_counting", "ties_in_lds_by_histogram", "ties_beyond_lds",
                                  "kth_far_above_threshold", "more_candidates_than_registers"])
def test_every_route_of_the_row_select(oracle, case):
    """Rows built to drive mv_row_select down each of its routes: crowded
    histogram bins (equal magnitudes), tie groups small / large / larger than the
    LDS list, a K-th magnitude more than an octave above the estimate, and a
    candidate list that needs the kernel's instance with more list entries per thread."""
    rng = np.random.default_rng(sum(map(ord, case)))
    N, d, K = 3, 300007, 3000
    if case == "ties_in_lds_by_counting":
        groups = [(2600, 2.0, 3.0), (900, 1.0, 1.0)]            # 900 ties, 400 taken
    elif case == "ties_in_lds_by_histogram":
        groups = [(2000, 2.0, 3.0), (5000, 1.0, 1.0)]           # 5000 ties, 1000 taken
    elif case == "ties_beyond_lds":
        groups = [(2000, 2.0, 3.0), (20000, 1.0, 1.0)]          # 20000 ties, 1000 taken
    elif case == "kth_far_above_threshold":
        groups = [(3500, 8.0, 16.0), (2600, 1.0, 1.1)]          # > K coordinates beyond 2 tau
    else:
        N, d, K = 2, 600011, 40000                              # about 46000 candidates per row
        groups = []
    say("select route %s N=%d d=%d K=%d" % (case, N, d, K))
    if groups:
        g = np.stack([_levels_row(rng, d, groups) for _ in range(N)])
    else:
        g = rng.standard_normal((N, d)).astype(np.float32)
    e = np.zeros_like(g)
    with GpuStepper(N, d, K) as gs:
        gs.set_error(e)
        gs.set_grads(g)
        gs.step()
        got = gs.fetch()
        cand, _, path = gs.row_stats()
    say("  candidates %s path %s" % (cand, path))
    assert_matches_oracle(got, oracle.vote_step(g, e, K), case)
    assert all(p != 1 for p in path), "these rows are meant for the candidate-list routes"
    if case == "kth_far_above_threshold":
        assert all(p == 2 for p in path)
    if case == "more_candidates_than_registers":
        assert min(cand) > 32768


@pytest.mark.parametrize("case", ["normal", "lattice_ties", "kth_far_above_threshold"])
def test_long_candidate_lists_are_selected_by_many_workgroups(oracle, case):
    """Candidate lists far longer than a workgroup of mv_row_select keeps in registers
    (32 x 1024 entries; about 240,000 per row here): selected, and their votes cast, by
    mv_sel_hist, mv_sel_split and mv_sel_finish, many workgroups per row."""
    rng = np.random.default_rng(sum(map(ord, case)))
    N, d, K = 3, 1500007, 220000
    if case == "normal":
        g = rng.standard_normal((N, d)).astype(np.float32)
    elif case == "lattice_ties":
        g = (np.round(rng.standard_normal((N, d)) * 24.0) / 64.0).astype(np.float32)   # about 200 distinct magnitudes
    else:
        g = np.stack([_levels_row(rng, d, [(240000, 8.0, 16.0), (150000, 1.0, 1.1)]) for _ in range(N)])
    e = np.zeros_like(g)
    say("many-workgroup select %s N=%d d=%d K=%d" % (case, N, d, K))
    with GpuStepper(N, d, K) as gs:
        gs.set_error(e)
        gs.set_grads(g)
        gs.step()
        got = gs.fetch()
        cand, _, path = gs.row_stats()
    say("  candidates %s path %s" % (cand, path))
    assert_matches_oracle(got, oracle.vote_step(g, e, K), case)
    assert all(p != 1 for p in path), "these rows are meant for the candidate-list routes"
    assert min(cand) > 160 * 1024, "these lists are meant to be far longer than one workgroup keeps"


def test_tie_cut_inside_a_run_of_neighbouring_ties(oracle):
    """6000 coordinates tie at the K-th magnitude; 1500 of them are neighbours at the
    start of a long row and the cut falls among these, so the narrowing by the
    coordinates' leading bits leaves more than a workgroup can rank by counting."""
    rng = np.random.default_rng(77)
    N, d, K = 2, 5000011, 30000
    g = np.empty((N, d), np.float32)
    for n in range(N):
        row = (rng.standard_normal(d) * 1e-3).astype(np.float32)
        far = 10000 + rng.permutation(d - 10000)
        row[far[:29000]] = rng.uniform(2.0, 3.0, 29000).astype(np.float32)
        row[far[29000:59000]] = rng.uniform(0.5, 0.9, 30000).astype(np.float32)
        row[far[59000:63500]] = 1.0
        row[100 + 7 * n:1600 + 7 * n] = -1.0                  # the neighbours; 1000 of them are taken
        g[n] = row
    e = np.zeros_like(g)
    say("tie cut among neighbouring ties N=%d d=%d K=%d" % (N, d, K))
    with GpuStepper(N, d, K) as gs:
        gs.set_error(e)
        gs.set_grads(g)
        gs.step()
        got = gs.fetch()
        cand, _, path = gs.row_stats()
    say("  candidates %s path %s" % (cand, path))
    assert all(p != 1 for p in path), "meant for the candidate-list routes"
    assert_matches_oracle(got, oracle.vote_step(g, e, K), "neighbouring ties")


@pytest.mark.parametrize("d,K", [(40009, 1), (40009, 400), (40009, 700), (40009, 1500), (40009, 33000),
                                 (400003, 300000)])
def test_one_worker_of_a_long_vector(oracle, d, K):
    """One worker: a round of the gather has 1024 positions, whose values and coordinates lie side by side in LDS; with
    a workgroup's positions below, at and far beyond a round, in all three schemes."""
    say("one worker d=%d K=%d" % (d, K))
    rng = np.random.default_rng(d + K)
    e = (rng.standard_normal((1, d)) * 0.1).astype(np.float32)
    with GpuStepper(1, d, K) as gs:
        gs.set_error(e)
        for t in range(4):
            g = rng.standard_normal((1, d)).astype(np.float32)
            gs.set_grads(g)
            if t % 2 == 0:
                gs.step()
                ref = oracle.vote_step(g, e, K, threads=8)
            else:
                r = rng.standard_exponential(d).astype(np.float32)
                gs.step_rs(r)
                ref = oracle.rs_vote_step(g, e, K, r, threads=8)
            assert_matches_oracle(gs.fetch(), ref, "step %d" % t)
            e = ref.err
    gs = GpuAdStepper(1, d, K, K)
    try:
        vote, msum, e = np.zeros((1, d), np.uint8), np.zeros(d, np.uint8), np.zeros((1, d), np.float32)
        for t, k_ad in enumerate([K, max(1, K // 10)]):
            g = rng.standard_normal((1, d)).astype(np.float32)
            ref = oracle.ad_vote_step(g, e, K, k_ad, vote, msum, threads=8)
            gs.step(g, k_ad)
            gs.compare(ref, "add-drop step %d" % t)
            vote, msum, e = ref.vote, ref.msum, ref.err
    finally:
        gs.close()
