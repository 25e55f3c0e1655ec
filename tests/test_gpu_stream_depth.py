"""int8 weights, up to 64 rows: the two depths of the stream kernel (16 chunks of weights on their way, or a few) at the edges of the rule that
picks one.  Integer sums: the bits of the 64-row tiles that the same rows get in a larger call."""
import numpy as np
import pytest
import torch

import essa_workloads as wl
from helpers import bf16_dev, candidate_sigmas, gpu_proj, oracle_proj, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_ins,d_out", [
    ((8192,), 72),                                         # two full bunches, few blocks: deep on one row block and on two
    ((7200,), 40),                                         # 30 chunks a wave: the second bunch two short
    ((3584, 4096), 4104),                                  # 258 blocks: deep on two row blocks only
    ((3584, 3300), 96),                                    # 13 chunks beside 14: neither is deep
    ((8192,), 4160),                                       # 130 blocks, two bunches: deep on one row block only
])
def test_stream_depths_same_bits(essa, d_ins, d_out):
    ctx = essa.Context(0)
    K, big = 4, 100
    rd = to_dev(np.random.default_rng(12).integers(0, K, big).astype(np.int32))
    items = []
    for i, d_in in enumerate(d_ins):
        p = wl.make_projection("t", d_in, d_out, 8, "int8", layer=25, proj=i)
        _, f = oracle_proj(p)
        items.append((gpu_proj(essa, ctx, p), bf16_dev(wl.make_x_bf16(big, d_in, x_id=90 + i)[0])) + tuple(to_dev(s) for s in candidate_sigmas(f, K, 0.05)))
    for flags in (0, essa.COMPUTE_W8A8):
        outs = {}
        for R in (big, 16, 17, 24, 32, 33, 40, 41, 64):
            print("stream depth: d_in=%s d_out=%d R=%d flags=%d" % (d_ins, d_out, R, flags), flush=True)
            Y = [torch.full((R, d_out), float("nan"), device="cuda") for _ in items]
            essa.essa_svdlora_forward_group(ctx, [(gp, X[:R].contiguous(), rd[:R].contiguous(), sA, sB, y) for (gp, X, sA, sB), y in zip(items, Y)], flags)
            outs[R] = Y
            assert all(torch.equal(y, b[:R]) for y, b in zip(Y, outs[big])), R
    for it in items:
        it[0].close()
    ctx.close()
