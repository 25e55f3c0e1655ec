"""GPU parity of the kernel that streams 4-bit weights at small row counts (one to four row blocks of 32).

It adds the quantisation groups up in the tile kernels' order, so a row has the same bits whichever of them took it; against the
oracle the repository's bars for the 16-bit fixed-point path apply."""
import numpy as np
import pytest
import torch

import essa_workloads as wl
import oracle as orc
from helpers import bf16_dev, candidate_sigmas, gpu_proj, oracle_proj, to_dev

pytestmark = pytest.mark.gpu

LIMB_RMS, LIMB_MAX = 1e-4, 1e-3


@pytest.mark.parametrize("d_in,d_out,r", [
    (128, 40, 5),         # one group, two channel blocks, the second mostly empty
    (1152, 328, 32),      # nine groups: one in the second round, three of padding
    (3584, 129, 16),      # 28 groups: half of the fourth round; odd width
    (8192, 96, 24),       # every round full
])
def test_q4_stream_rows(essa, d_in, d_out, r):
    ctx = essa.Context(0)
    K, big = 5, 150
    print("q4 stream: d_in=%d d_out=%d r=%d" % (d_in, d_out, r), flush=True)
    p = wl.make_projection("t", d_in, d_out, r, "int4", layer=13, proj=2)
    W, f = oracle_proj(p)
    gp = gpu_proj(essa, ctx, p)
    sA, sB = candidate_sigmas(f, K, 0.05)
    sAd, sBd = to_dev(sA), to_dev(sB)
    xb, xv = wl.make_x_bf16(big, d_in, x_id=61)
    xb[2], xv[2] = 0, 0
    r2c = np.random.default_rng(9).integers(0, K, big).astype(np.int32)
    Xd, rd = bf16_dev(xb), to_dev(r2c)
    v = torch.randn(d_out, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
    nblk = (d_out + 127) // 128
    for flags, ref in ((0, orc.svdlora_forward(W, f, xv, r2c, sA, sB)), (essa.BASE_ONLY, xv.astype(np.float64) @ W.T),
                       (essa.LORA_ONLY, orc.svdlora_forward(W, f, xv, r2c, sA, sB, lora_only=True))):
        big32 = torch.empty(big, d_out, device="cuda")
        big16 = torch.empty(big, d_out, device="cuda", dtype=torch.bfloat16)
        essa.essa_svdlora_forward(ctx, gp, Xd, rd, sAd, sBd, big32, flags)          # 150 rows: the tile kernels
        essa.essa_svdlora_forward(ctx, gp, Xd, rd, sAd, sBd, big16, flags)
        for R in (1, 16, 32, 33, 96, 97, 128, 129):
            for start in (0, big - R):
                sub = slice(start, start + R)
                Xs, rs = Xd[sub].contiguous(), rd[sub].contiguous()
                Y32 = torch.full((R, d_out), float("nan"), device="cuda")
                Y16 = torch.full((R, d_out), float("nan"), device="cuda", dtype=torch.bfloat16)
                rowpart = torch.full((nblk, R), float("nan"), device="cuda")
                essa.essa_svdlora_forward_reward_group(ctx, [(gp, Xs, rs, sAd, sBd, Y32)], [v], rowpart, 0, flags)
                essa.essa_svdlora_forward(ctx, gp, Xs, rs, sAd, sBd, Y16, flags)
                assert torch.equal(Y32, big32[sub]) and torch.equal(Y16, big16[sub]), (flags, R, start)
                e_max, e_rms = orc.rel_errors(Y32.cpu().numpy(), ref[sub])
                assert e_rms <= LIMB_RMS and e_max <= LIMB_MAX, (flags, R, start, e_max, e_rms)
                # the partials are sums of 128 products of the outputs as written, in fp32
                pad = torch.zeros(R, nblk * 128 - d_out, device="cuda", dtype=torch.float64)
                want = torch.cat([Y32.double() * v.double(), pad], 1).view(R, nblk, 128)
                assert torch.all((rowpart.T.double() - want.sum(2)).abs() <= 128 * 2.0 ** -24 * want.abs().sum(2) + 1e-30)
    # a non-finite entry spoils its own row and nothing else
    good, bad = torch.empty(20, d_out, device="cuda"), torch.empty(20, d_out, device="cuda")
    Xs, rs = Xd[:20].clone(), rd[:20].contiguous()
    essa.essa_svdlora_forward(ctx, gp, Xs, rs, sAd, sBd, good)
    Xs[7, d_in - 1] = float("inf")
    essa.essa_svdlora_forward(ctx, gp, Xs, rs, sAd, sBd, bad)
    keep = torch.arange(20, device="cuda") != 7
    assert torch.isnan(bad[7]).all() and torch.equal(bad[keep], good[keep])
    gp.close()
    ctx.close()


def test_q4_stream_grouped_mixed_rows(essa):
    """Items of different row counts and ranks in one call: each item alone gives the same bits."""
    ctx = essa.Context(0)
    d_in, K = 640, 4
    items = []
    for i, (d_out, r, R) in enumerate(((200, 16, 25), (96, 8, 25), (328, 32, 50), (64, 4, 64))):
        p = wl.make_projection("t", d_in, d_out, r, "int4", layer=19, proj=i)
        _, f = oracle_proj(p)
        sA, sB = candidate_sigmas(f, K, 0.05, pert_id=i)
        xb, _ = wl.make_x_bf16(R, d_in, x_id=80 + R)
        r2c = np.random.default_rng(R).integers(0, K, R).astype(np.int32)
        items.append((gpu_proj(essa, ctx, p), bf16_dev(xb), to_dev(r2c), to_dev(sA), to_dev(sB), torch.empty(R, d_out, device="cuda")))
    essa.essa_svdlora_forward_group(ctx, items)
    for it in items:
        Y1 = torch.empty_like(it[5])
        essa.essa_svdlora_forward(ctx, *it[:5], Y1)
        assert torch.equal(Y1, it[5])
        it[0].close()
    ctx.close()
