"""A generation of a small search: candidates in one launch (up to 64 dimensions), the rows' reward sums inside the candidates' means (up to 16 blocks)."""
import numpy as np
import pytest
import torch

import oracle as orc
from helpers import seeds_dev, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 7, 16, 63, 64, 65])            # 65: the two launches
@pytest.mark.parametrize("K", [1, 15, 16, 17, 40])
def test_small_sampler(essa, n, K):
    g = np.random.default_rng(100 * n + K)
    ctx = essa.Context(0)
    cma = essa.CmaState(ctx, n, 0.32, g.standard_normal(n).astype(np.float32))
    B, d = g.standard_normal((n, n)).astype(np.float32), g.uniform(0.5, 2.0, n).astype(np.float32)
    cma.set_basis(to_dev(B), to_dev(d))
    seeds = g.integers(0, 2 ** 32, K, dtype=np.uint32)
    theta, z = torch.full((K, n), float("nan"), device="cuda"), torch.full((K, n), float("nan"), device="cuda")
    essa.essa_sample_candidates(ctx, cma, seeds_dev(seeds), theta, z)
    again = torch.empty_like(theta)
    essa.essa_sample_candidates(ctx, cma, seeds_dev(seeds), again)
    st = cma.export()
    ref, ref_z = orc.sample_candidates(st["m"].astype(np.float64), np.float32(0.32), B.astype(np.float64), d.astype(np.float64), [int(s) for s in seeds])
    assert torch.equal(theta, again)
    assert orc.rel_errors(z.cpu().numpy(), ref_z)[1] <= 1e-6
    # fp32 sums of n terms of mixed sign: n 2^-24 of the sum of their magnitudes at most
    mag = np.abs(st["m"]) + 0.32 * np.abs(d * ref_z) @ np.abs(B).T
    assert np.all(np.abs(theta.cpu().numpy() - ref) <= (n + 4) * 2.0 ** -24 * mag + 1e-7 * np.abs(ref))
    cma.close()
    ctx.close()


@pytest.mark.parametrize("blocks", [1, 2, 15, 16, 17])                 # 17: a launch of its own for the rows' sums
@pytest.mark.parametrize("R,K", [(1, 1), (70, 3), (300, 5)])
def test_reward_finish_few_blocks(essa, blocks, R, K):
    g = np.random.default_rng(blocks + R)
    ctx = essa.Context(0)
    part = g.standard_normal((blocks, R)).astype(np.float32)
    r2c = np.arange(R, dtype=np.int32) % K
    F0 = g.standard_normal(K).astype(np.float32)
    F = to_dev(F0)
    essa.essa_reward_finish(ctx, to_dev(part), blocks, to_dev(r2c), F)
    rows = part.astype(np.float64).sum(0)
    want = np.array([rows[r2c == k].mean() for k in range(K)])
    # fp64 sums, one rounding to fp32 and one of the addition to F
    assert np.all(np.abs(F.cpu().numpy() - (F0 + want)) <= 2.0 ** -23 * (np.abs(F0) + np.abs(want)) + 1e-12)
    ctx.close()


# the map is read 1024 places at a time, four a thread: around that, and many rows of few candidates
@pytest.mark.parametrize("blocks", [1, 2, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("R,K", [(255, 2), (1023, 1), (1025, 3), (5000, 1), (5000, 40)])
def test_reward_finish_one_launch_has_the_bits_of_two(essa, blocks, R, K):
    g = np.random.default_rng(1000 * blocks + R + K)
    ctx = essa.Context(0)
    part = np.zeros((17, R), np.float32)                   # blocks of zeros behind the last one take the two launches and change no sum
    part[:blocks] = g.standard_normal((blocks, R))
    r2c = g.integers(0, K, R).astype(np.int32)
    r2c[:K] = np.arange(K)
    F = [torch.zeros(K, device="cuda") for _ in range(2)]
    for out, count in zip(F, (blocks, 17)):
        essa.essa_reward_finish(ctx, to_dev(part), count, to_dev(r2c), out)
    rows = part.astype(np.float64).sum(0)
    want = np.array([rows[r2c == k].mean() for k in range(K)])
    assert torch.equal(F[0].view(torch.int32), F[1].view(torch.int32))
    # fp64 sums of R terms at most, one rounding to fp32
    assert np.all(np.abs(F[0].cpu().numpy() - want) <= 2.0 ** -24 * np.abs(want) + 1e-12)
    ctx.close()


def test_reward_finish_few_candidates_many_rows_take_no_longer_in_one_launch(essa):
    """16 blocks of 32768 rows of one candidate: all of it is one workgroup's work.  17 blocks are two launches and more to read."""
    R = 32768
    ctx = essa.Context(0)
    part, r2c, F = torch.randn(17, R, device="cuda"), torch.zeros(R, dtype=torch.int32, device="cuda"), torch.zeros(1, device="cuda")

    def us(blocks):
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                essa.essa_reward_finish(ctx, part, blocks, r2c, F)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 50)
        return best

    us(17)
    one, two = us(16), us(17)
    print("one launch %.1f us, two %.1f us" % (one, two), flush=True)
    assert one <= 1.5 * two                                # 47 and 53; with a wait for every partial and place 207 and 69
    ctx.close()


# 4, 8 or 16 candidates a workgroup: up to 32 dimensions 8 as long as there are at most 1024 such workgroups, from 33 on 4, else 16
@pytest.mark.parametrize("n,K", [(16, 33), (17, 9), (17, 8193), (32, 8192), (33, 5), (33, 4097), (64, 4095), (64, 4097)])
def test_small_sampler_candidates_do_not_hang_on_their_workgroup(essa, n, K):
    g = np.random.default_rng(n + K)
    ctx = essa.Context(0)
    cma = essa.CmaState(ctx, n, 0.32, g.standard_normal(n).astype(np.float32))
    cma.set_basis(to_dev(g.standard_normal((n, n)).astype(np.float32)), to_dev(g.uniform(0.5, 2.0, n).astype(np.float32)))
    seeds = seeds_dev(g.integers(0, 2 ** 32, K, dtype=np.uint32))
    theta, z = torch.full((K, n), float("nan"), device="cuda"), torch.full((K, n), float("nan"), device="cuda")
    essa.essa_sample_candidates(ctx, cma, seeds, theta, z)
    for lo in range(0, K, 999):
        hi = min(lo + 999, K)
        t, zz = torch.empty(hi - lo, n, device="cuda"), torch.empty(hi - lo, n, device="cuda")
        essa.essa_sample_candidates(ctx, cma, seeds[lo:hi].clone(), t, zz)
        assert torch.equal(theta[lo:hi], t) and torch.equal(z[lo:hi], zz)
    cma.close()
    ctx.close()


def test_small_sampler_many_candidates_of_few_dimensions(essa):
    """Up to 16 dimensions more than 24576 candidates go in two launches: the same normals, sums of n terms in another order."""
    n, K = 16, 24577
    g = np.random.default_rng(7)
    ctx = essa.Context(0)
    B, d = g.standard_normal((n, n)).astype(np.float32), g.uniform(0.5, 2.0, n).astype(np.float32)
    cma = essa.CmaState(ctx, n, 0.32)
    cma.set_basis(to_dev(B), to_dev(d))
    seeds = seeds_dev(g.integers(0, 2 ** 32, K, dtype=np.uint32))
    out = [[torch.full((k, n), float("nan"), device="cuda") for _ in range(2)] for k in (K, K - 1)]
    for (theta, z), k in zip(out, (K, K - 1)):
        essa.essa_sample_candidates(ctx, cma, seeds[:k].clone(), theta, z)
    assert torch.equal(out[0][1][:-1], out[1][1])
    z = out[0][1].double().cpu().numpy()
    ref, mag = 0.32 * (z * d) @ B.T.astype(np.float64), 0.32 * np.abs(z * d) @ np.abs(B).T
    for theta, _ in out:                                   # fp32 sums of n terms of mixed sign: n 2^-24 of the sum of their magnitudes at most
        assert np.all(np.abs(theta.cpu().numpy() - ref[:len(theta)]) <= (n + 4) * 2.0 ** -24 * mag[:len(theta)])
    cma.close()
    ctx.close()


def test_small_sampler_takes_no_longer_than_two_launches(essa):
    """Replayed in turn: 64 dimensions in one launch against 65 in two."""
    runs, times = {}, {}
    for n in (64, 65):
        stream = torch.cuda.Stream()
        ctx = essa.Context(0, stream)
        cma = essa.CmaState(ctx, n, 0.32)
        seeds, theta = torch.arange(32, dtype=torch.int32, device="cuda"), torch.empty(32, n, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            essa.essa_sample_candidates(ctx, cma, seeds, theta)
            ctx.graph_begin()
            for _ in range(20):
                essa.essa_sample_candidates(ctx, cma, seeds, theta)
            runs[n] = (stream, ctx.graph_end(), ctx, cma, seeds, theta)
    for _ in range(40):
        for n, (stream, graph, *_) in runs.items():
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            with torch.cuda.stream(stream):
                a.record(stream)
                graph.launch()
                b.record(stream)
            stream.synchronize()
            times[n] = min(times.get(n, float("inf")), a.elapsed_time(b) * 50)
    for _, graph, ctx, cma, *_ in runs.values():
        graph.close()
        cma.close()
        ctx.close()
    print(times, flush=True)
    assert times[64] <= times[65]                          # 5.7 and 7.1 us; with 16 candidates a workgroup 7.9
