"""Short vectors (up to 32,768 coordinates), which take a way of their own: all three kinds of step against the
oracle, element by element, at the edges of the coordinates per thread (4096, 8192, 16384, 32768), of the bitmaps'
words, of the rounds of mask positions per workgroup and of the votes' bits, and with the values that drive the row
select down each of its routes."""
import sys

import numpy as np
import pytest
import torch

from tests.gpu_util import GpuStepper, assert_matches_oracle
from tests.test_gpu_add_drop import GpuAdStepper

pytestmark = pytest.mark.gpu


def values(rng, kind, N, d):
    if kind == "normal":
        g = rng.standard_normal((N, d))
    elif kind == "lattice":          # a few magnitudes, most of them zero: ties, also of zeros
        g = np.round(rng.standard_normal((N, d)) * 0.6) / 8
    elif kind == "equal":            # one magnitude
        g = rng.choice([-1.5, 1.5], (N, d))
    elif kind == "crowded":          # thousands of distinct magnitudes with the same 13 leading bits
        g = 1.0 + rng.random((N, d)) * 2.0 ** -6
    else:                            # "one_bin": the top K are exactly the members of the highest bins
        g = rng.standard_normal((N, d)) * 1e-3
        g[:, :: max(1, d // 40)] = 7.0
    return g.astype(np.float32)


CASES = [(1, 1, 1, "normal"), (3, 31, 31, "lattice"), (2, 33, 7, "normal"), (5, 4095, 40, "normal"),
         (4, 4096, 41, "lattice"), (2, 4097, 4097, "normal"), (7, 8192, 82, "crowded"), (16, 8193, 300, "normal"),
         (4, 10007, 101, "equal"), (3, 10007, 41, "one_bin"), (31, 16384, 164, "normal"), (32, 16385, 20, "lattice"),
         (2, 32767, 9000, "crowded"), (40, 32768, 546, "normal"), (255, 20011, 200, "lattice"), (128, 5000, 4100, "normal"),
         (3, 32769, 300, "normal")]


@pytest.mark.parametrize("N,d,K,kind", CASES)
@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
def test_short_vectors(oracle, N, d, K, kind, bf16):
    print("[case] short vectors N=%d d=%d K=%d %s bf16=%s" % (N, d, K, kind, bf16), flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(N * 100_000 + d + K)

    def grads():
        g = values(rng, kind, N, d)
        return torch.from_numpy(g).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16) if bf16 else g

    e = np.zeros((N, d), np.float32)
    with GpuStepper(N, d, K, bf16=bf16, extra_ld=1) as gs:     # plain and random steps share the context
        gs.set_error(e)
        for t in range(4):
            g = grads()
            gs.set_grads(g)
            if t % 2 == 0:
                gs.step()
                ref = oracle.vote_step(g, e, K, threads=8)
            else:
                r = rng.standard_exponential(d).astype(np.float32)
                r = np.round(r * 2) / 2 if t == 3 else r              # equal times, zeros among them
                gs.step_rs(r)
                ref = oracle.rs_vote_step(g, e, K, r, threads=8)
            assert_matches_oracle(gs.fetch(), ref, "step %d" % t)
            e = ref.err
        cand, tau, path = gs.row_stats()
        if d <= 32768:
            assert set(cand) == {d} and set(tau) == {0} and set(path) == {0}
    gs = GpuAdStepper(N, d, K, K, bf16=bf16)
    try:
        vote, msum, e = np.zeros((N, d), np.uint8), np.zeros(d, np.uint8), np.zeros((N, d), np.float32)
        for t, k_ad in enumerate([max(1, K // 3), K, max(1, K // 9), 1]):
            g = grads()
            ref = oracle.ad_vote_step(g, e, K, k_ad, vote, msum, threads=8)
            gs.step(g, k_ad)
            gs.compare(ref, "add-drop step %d k_ad %d" % (t, k_ad))
            vote, msum, e = ref.vote, ref.msum, ref.err
    finally:
        gs.close()


@pytest.mark.parametrize("scheme", ["plain", "random"])
def test_captured_short_step_replays(oracle, scheme):
    """A captured step replayed several times with eager steps in between gives the eager results."""
    N, d, K = 5, 9001, 90
    print("[case] captured short step %s" % scheme, flush=True)
    rng = np.random.default_rng(5)
    r = rng.standard_exponential(d).astype(np.float32)
    r_dev = torch.from_numpy(r).to("cuda:0")
    with GpuStepper(N, d, K) as gs:
        from paper_2011_06495_amd import binding as B

        def enqueue():
            if scheme == "plain":
                gs.step()
            else:
                B.mv_rs_vote_step(gs.ctx, gs.g, gs.e, r_dev, gs.widx, gs.votes, gs.mask, gs.agg, ld_g=gs.ld_g,
                                  ld_e=gs.ld_e)

        e = np.zeros((N, d), np.float32)
        gs.set_error(e)
        gs.set_grads(values(rng, "normal", N, d))
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            enqueue()
        for t in range(5):
            g = values(rng, "normal", N, d)
            gs.set_grads(g)
            torch.cuda.synchronize()
            if t == 2:
                enqueue()
            else:
                graph.replay()
            ref = oracle.vote_step(g, e, K) if scheme == "plain" else oracle.rs_vote_step(g, e, K, r)
            assert_matches_oracle(gs.fetch(), ref, "%s step %d" % (scheme, t))
            e = ref.err


@pytest.mark.parametrize("kind", ["normal", "lattice", "equal"])
@pytest.mark.parametrize("N,d,K", [(3, 32769, 3), (2, 262145, 2600), (2, 524288, 100), (2, 524289, 100),
                                   (2, 524320, 524320), (1, 1 << 20, 10486), (2, (1 << 20) + 1, 10486)])
def test_rows_sampled_by_one_workgroup(oracle, kind, N, d, K):
    """Beyond the short vectors a row's threshold is estimated by one workgroup up to a size that depends on K, then
    by several: both sides of the lines, with K from a handful to all of the row."""
    print("[case] one sampling workgroup N=%d d=%d K=%d %s" % (N, d, K, kind), flush=True)
    rng = np.random.default_rng(d + K)
    e = np.zeros((N, d), np.float32)
    with GpuStepper(N, d, K) as gs:
        gs.set_error(e)
        for t in range(2):
            g = values(rng, kind, N, d)
            gs.set_grads(g)
            gs.step()
            ref = oracle.vote_step(g, e, K, threads=8)
            assert_matches_oracle(gs.fetch(), ref, "%s step %d" % (kind, t))
            e = ref.err


@pytest.mark.parametrize("kind", ["normal", "lattice"])
@pytest.mark.parametrize("N,d,K", [(3, 1150003, 11500), (2, 1200007, 12000), (2, 1200007, 13500), (2, 1200007, 6000)])
def test_longer_rows_sampled_by_one_workgroup(oracle, kind, N, d, K):
    """Rows beyond 2^20 coordinates whose lists are short enough for one sampling workgroup, and such whose are not:
    too long, and too long against what several sampling workgroups would give."""
    print("[case] longer rows, one sampling workgroup N=%d d=%d K=%d %s" % (N, d, K, kind), flush=True)
    rng = np.random.default_rng(d + K)
    e = np.zeros((N, d), np.float32)
    with GpuStepper(N, d, K) as gs:
        gs.set_error(e)
        for t in range(2):
            g = values(rng, kind, N, d)
            gs.set_grads(g)
            gs.step()
            ref = oracle.vote_step(g, e, K, threads=8)
            assert_matches_oracle(gs.fetch(), ref, "%s step %d" % (kind, t))
            e = ref.err
