"""GPU parity of the update's right-hand sides (ranking, regenerated normals, their weighted sum): one launch for up to 64 of them, 32 at a
time, kernels of their own beyond; the ranking inside up to 256 candidates.  At the edges of each, against the oracle's step."""
import numpy as np
import pytest
import torch

import oracle as orc
from helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,K", [(1, 2), (16, 64), (17, 65), (66, 66), (260, 128), (67, 130), (63, 256), (130, 258), (65, 300)])
def test_update_right_hand_sides(essa, n, K):
    ctx = essa.Context(0)
    print("n=%d K=%d" % (n, K), flush=True)
    g = np.random.default_rng(1000 * n + K)
    seeds = list(range(7, 7 + K))
    F = g.standard_normal(K).astype(np.float32)
    if K > 4:
        F[K // 2] = F[1]                                   # a tie: ascending index
        F[2] = np.nan                                      # ranks last
    cma = essa.CmaState(ctx, n, 0.32, None)
    order = torch.full((K,), -1, dtype=torch.int32, device="cuda")
    essa.essa_cmaes_update(ctx, cma, to_dev(np.array(seeds, np.int32)), to_dev(F), order)
    st, want_order = orc.cma_update(orc.cma_state_init(n, np.float32(0.32)), seeds, F)
    assert np.array_equal(order.cpu().numpy(), want_order)
    got = cma.export()
    # fp32 sums over n of fp64-rounded terms; the repository's bar for the update
    for name in ("m", "p_sigma", "p_c", "C"):
        assert orc.rel_errors(got[name], getattr(st, name))[1] <= 1e-5, name
    # the same without the order asked for
    again = essa.CmaState(ctx, n, 0.32, None)
    essa.essa_cmaes_update(ctx, again, to_dev(np.array(seeds, np.int32)), to_dev(F))
    assert np.array_equal(again.export()["C"], got["C"])
    again.close()
    cma.close()
    ctx.close()


@pytest.mark.parametrize("kind,n,K", [("OPT_CMA", 700, 32), ("OPT_CMA", 130, 300), ("OPT_CMA", 66, 1024), ("OPT_ACTIVE_CMA", 200, 40), ("OPT_ACTIVE_CMA", 67, 260),
                                      ("OPT_SEP_CMA", 1500, 48), ("OPT_SEP_CMA", 50, 270), ("OPT_ES", 300, 32), ("OPT_ES", 70, 260), ("OPT_ARS", 90, 40)])
def test_order_out_over_an_input(essa, kind, n, K):
    """The ranking may be written over the rewards or the seeds: every launch of the update that reads them comes first."""
    print("%s n=%d K=%d" % (kind, n, K), flush=True)
    ctx = essa.Context(0)
    g = np.random.default_rng(n + K)
    F = g.standard_normal(K).astype(np.float32)
    ars = kind == "OPT_ARS"                                # one seed and one place in the order per pair
    S = K // 2 if ars else K
    results = []
    for over in (None, "rewards", "seeds"):
        cma = essa.CmaState(ctx, n, 0.32, kind=getattr(essa, kind), ars_alpha=0.02 if ars else 0.0, ars_top=8 if ars else 0)
        seeds, rewards = to_dev(np.arange(5, 5 + S, dtype=np.int32)), to_dev(F)
        order = torch.full((S,), -1, dtype=torch.int32, device="cuda") if over is None else rewards.view(torch.int32)[:S] if over == "rewards" else seeds
        essa.essa_cmaes_update(ctx, cma, seeds, rewards, order)
        state = cma.export()
        results.append([order.cpu().numpy()] + [np.asarray(state[k]) for k in sorted(state)])
        cma.close()
    want = np.argsort(-(np.maximum(F[::2], F[1::2]) if ars else F), kind="stable")
    for r in results:
        assert np.array_equal(r[0], want)
        assert all(np.array_equal(a, b) for a, b in zip(r, results[0]))
    ctx.close()


def _scratch_of(essa, ctx, rows):
    """The context's first scratch: five quarters of 4 bytes a row and a megabyte, pinned by a recorded graph."""
    Y, v = torch.zeros(rows, 1, device="cuda"), torch.zeros(1, device="cuda")
    essa.essa_reward_accumulate(ctx, Y, v, torch.zeros(rows, dtype=torch.int32, device="cuda"), torch.zeros(1, device="cuda"))
    sft = torch.ones(1, 2, device="cuda")
    theta, out = torch.zeros(1, 4, device="cuda"), (torch.empty(1, 1, 2, device="cuda"), torch.empty(1, 1, 2, device="cuda"))
    torch.cuda.synchronize()
    ctx.graph_begin()
    essa.essa_theta_to_sigma(ctx, 2, sft, sft, theta, *out)
    return ctx.graph_end()


@pytest.mark.parametrize("what,n,K,rows", [
    ("sample", 15400, 17, 64),                             # a megabyte of scratch for 17 rows: one tile of 16 at a time
    ("sample", 5, 65536, 100000),                          # five columns in tiles of 16: some candidates at a time
    ("update", 10000, 8, 64),                              # 6 right-hand sides and what comes of them
    ("update", 401, 300, 64),                              # the launches for more than 64 right-hand sides
])
def test_scratch_that_cannot_grow(essa, what, n, K, rows):
    """Calls whose rows fit a scratch that a recorded graph pins go through (three times a right-hand side of n floats for an update, one per candidate
    for the sampler), with the bits of a context that is free to grow."""
    print("%s n=%d K=%d" % (what, n, K), flush=True)
    got = []
    for pinned in (False, True):
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            ctx = essa.Context(0, side)
            graph = _scratch_of(essa, ctx, rows) if pinned else None
            cma = essa.CmaState(ctx, n, 0.32)
            seeds = to_dev(np.arange(3, 3 + K, dtype=np.int32))
            if what == "sample":
                theta, z = torch.empty(K, n, device="cuda"), torch.empty(K, n, device="cuda")
                essa.essa_sample_candidates(ctx, cma, seeds, theta, z)
                side.synchronize()
                got.append([theta.cpu().numpy(), z.cpu().numpy()])
            else:
                essa.essa_cmaes_update(ctx, cma, seeds, to_dev(np.random.default_rng(n).standard_normal(K).astype(np.float32)))
                side.synchronize()
                state = cma.export()
                got.append([state[k] for k in ("m", "p_sigma", "p_c", "C")])
            if graph is not None:
                graph.close()
            cma.close()
            ctx.close()
    assert all(np.array_equal(a, b) for a, b in zip(*got))
