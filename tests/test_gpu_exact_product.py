"""GPU parity of the exact-product kernel (int8 weights as bf16, fp32 accumulation) at the edges of its tiles and K steps.

Its products are exact; what is left is fp32 accumulation (one rounding of 2^-24 per 32 columns of a random-sign sum:
2^-24 sqrt(d_in / 32), 1e-6 at the widest row here) and the bf16 head + tail operands of the rank-r term (2^-17 of a term that is
a twentieth of the output), so the repository's bar for exact products applies, and a tenth of it to the base term alone."""
import numpy as np
import pytest
import torch

import essa_workloads as wl
import oracle as orc
from helpers import bf16_dev, bf16_host, candidate_sigmas, gpu_proj, oracle_proj, to_dev

pytestmark = pytest.mark.gpu

EXACT_RMS, EXACT_MAX = 2e-5, 2e-4
BF16_RMS, BF16_MAX = 1e-3, 2e-2


@pytest.mark.parametrize("R,d_in,d_out,r,flags", [
    (1, 48, 129, 5, 8),            # one row, less than one K step, asked for by the flag
    (129, 64, 128, 32, 8),         # exactly one K step and one tile of channels, one row past a tile
    (513, 1040, 300, 32, 0),       # taken by itself, K ends 16 columns into a step
    (1030, 528, 9001, 16, 0),      # 160 x 256 tiles, odd output width (element-wise stores)
    (700, 2064, 8200, 16, 0),      # 256 x 128 tiles
    (2050, 4112, 5000, 24, 0),     # 192 x 256 tiles, ragged rows and channels
])
def test_exact_product_tiles(essa, R, d_in, d_out, r, flags):
    ctx = essa.Context(0)
    K = 3
    print("exact product: R=%d d_in=%d d_out=%d r=%d" % (R, d_in, d_out, r), flush=True)
    p = wl.make_projection("t", d_in, d_out, r, "int8", layer=11, proj=1)
    p.scales[d_out // 2] = 0.0                             # a channel that has no base term at all
    W, f = oracle_proj(p)
    gp = gpu_proj(essa, ctx, p)
    sA, sB = candidate_sigmas(f, K, 0.05)
    xb, xv = wl.make_x_bf16(R, d_in, x_id=31)
    r2c = np.random.default_rng(6).integers(0, K, R).astype(np.int32)
    ref = orc.svdlora_forward(W, f, xv, r2c, sA, sB)
    Xd, rd, sAd, sBd = bf16_dev(xb), to_dev(r2c), to_dev(sA), to_dev(sB)
    v = torch.randn(d_out, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    nblk = (d_out + 127) // 128
    for dtype in (torch.float32, torch.bfloat16):
        Y = torch.full((R, d_out), float("nan"), device="cuda", dtype=dtype)
        rowpart = torch.full((nblk, R), float("nan"), device="cuda")
        essa.essa_svdlora_forward_reward_group(ctx, [(gp, Xd, rd, sAd, sBd, Y)], [v], rowpart, 0, flags)
        if dtype == torch.float32:
            e_max, e_rms = orc.rel_errors(Y.cpu().numpy(), ref)
            assert e_rms <= EXACT_RMS and e_max <= EXACT_MAX, (e_rms, e_max)
        else:
            e_max, e_rms = orc.rel_errors(bf16_host(Y), orc.round_to_bf16(ref))
            assert e_rms <= BF16_RMS and e_max <= BF16_MAX, (e_rms, e_max)
        # the partials are sums of 128 products of the outputs as written, in fp32
        pad = torch.zeros(R, nblk * 128 - d_out, device="cuda", dtype=torch.float64)
        want = (torch.cat([Y.double() * v.double(), pad], 1)).view(R, nblk, 128)
        assert torch.all((rowpart.T.double() - want.sum(2)).abs() <= 128 * 2.0 ** -24 * want.abs().sum(2) + 1e-30)
    Y = torch.empty(R, d_out, device="cuda")
    essa.essa_svdlora_forward(ctx, gp, Xd, rd, sAd, sBd, Y, flags | essa.BASE_ONLY)
    e_max, e_rms = orc.rel_errors(Y.cpu().numpy(), orc.svdlora_forward(W, f, xv, r2c, sA, sB, base_only=True))
    assert e_rms <= EXACT_RMS / 10 and e_max <= EXACT_MAX / 10, (e_rms, e_max)
    # a non-finite entry spoils its own row and nothing else
    Xbad = Xd.clone()
    Xbad[R // 2, d_in - 1] = float("inf")
    Ybad, Y = torch.empty(R, d_out, device="cuda"), torch.empty(R, d_out, device="cuda")
    essa.essa_svdlora_forward(ctx, gp, Xbad, rd, sAd, sBd, Ybad, flags)
    essa.essa_svdlora_forward(ctx, gp, Xd, rd, sAd, sBd, Y, flags)
    keep = torch.arange(R, device="cuda") != R // 2
    assert torch.isnan(Ybad[R // 2]).all() and torch.equal(Ybad[keep], Y[keep])
    # nor does the base term alone leave infinities in it
    essa.essa_svdlora_forward(ctx, gp, Xbad, rd, sAd, sBd, Ybad, flags | essa.BASE_ONLY)
    essa.essa_svdlora_forward(ctx, gp, Xd, rd, sAd, sBd, Y, flags | essa.BASE_ONLY)
    assert torch.isnan(Ybad[R // 2]).all() and torch.equal(Ybad[keep], Y[keep])
    gp.close()
    ctx.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_grouped_and_single_calls_agree(essa, dtype):
    """Which tile a projection gets hangs on its group (here 192 x 256 together, narrower ones alone); its outputs and reward
    partials do not, to the bit.  Ranks 16 and 32 in one launch, odd widths."""
    ctx = essa.Context(0)
    R, K, d_in = 1187, 5, 3584
    specs = [(3584, 16), (520, 32), (513, 7), (3600, 24)]
    Xs = [bf16_dev(wl.make_x_bf16(R, d_in, x_id=60 + i)[0]) for i in range(2)]
    rd = to_dev(np.random.default_rng(8).integers(0, K, R).astype(np.int32))
    items, vecs = [], []
    for i, (d_out, r) in enumerate(specs):
        p = wl.make_projection("t", d_in, d_out, r, "int8", layer=14, proj=i)
        _, f = oracle_proj(p)
        sA, sB = candidate_sigmas(f, K, 0.05, i)
        items.append([gpu_proj(essa, ctx, p), Xs[i == 3], rd, to_dev(sA), to_dev(sB), torch.empty(R, d_out, device="cuda", dtype=dtype)])
        vecs.append(torch.randn(d_out, device="cuda", generator=torch.Generator(device="cuda").manual_seed(i)))
    blocks = [(d_out + 127) // 128 for d_out, _ in specs]
    together = torch.full((sum(blocks), R), float("nan"), device="cuda")
    essa.essa_svdlora_forward_reward_group(ctx, [tuple(it) for it in items], vecs, together, 0)
    at = 0
    for it, v, nb in zip(items, vecs, blocks):
        Y, alone = torch.empty_like(it[5]), torch.full((nb, R), float("nan"), device="cuda")
        essa.essa_svdlora_forward_reward_group(ctx, [tuple(it[:5]) + (Y,)], [v], alone, 0)
        print("d_out=%d" % it[0].d_out, flush=True)
        assert torch.equal(Y, it[5])
        assert torch.equal(alone, together[at:at + nb])
        at += nb
    for it in items:
        it[0].close()
    ctx.close()


@pytest.mark.parametrize("r,flags,dtype", [(7, 0, torch.bfloat16), (24, 0, torch.float32), (16, 8, torch.float32), (32, 8, torch.bfloat16)])
def test_row_counts_that_change_the_tile(essa, r, flags, dtype):
    """1000 rows take the 64 x 128 tile, which forms u itself, 2000 the 128 x 128 one with five stages, 3700 the 160 x 128 one, 900
    without reward vectors the 64 x 64 one: the rows that they share have the same bits, outputs and reward partials, with and
    without the rank-r term."""
    ctx = essa.Context(0)
    K, d_in, d_out, Rs = 5, 1040, 1050, (1000, 2000, 3700)
    p = wl.make_projection("t", d_in, d_out, r, "int8", layer=18, proj=1)
    W, f = oracle_proj(p)
    gp = gpu_proj(essa, ctx, p)
    sA, sB = candidate_sigmas(f, K, 0.05)
    xb, xv = wl.make_x_bf16(Rs[-1], d_in, x_id=64)
    X, v = bf16_dev(xb), torch.randn(d_out, device="cuda")
    r2c = np.random.default_rng(6).integers(0, K, Rs[-1]).astype(np.int32)
    rd, sAd, sBd = to_dev(r2c), to_dev(sA), to_dev(sB)
    for more in (0, essa.BASE_ONLY):
        got = []
        for R in Rs:
            print("r=%d flags=%d R=%d" % (r, flags | more, R), flush=True)
            Y = torch.full((R, d_out), float("nan"), device="cuda", dtype=dtype)
            part = torch.full(((d_out + 127) // 128, R), float("nan"), device="cuda")
            essa.essa_svdlora_forward_reward_group(ctx, [(gp, X[:R], rd[:R], sAd, sBd, Y)], [v], part, 0, flags | more)
            got.append((Y[:Rs[0]], part[:, :Rs[0]]))
        for Y, part in got[1:]:
            assert torch.equal(Y, got[0][0]) and torch.equal(part, got[0][1])
        Y = torch.full((900, d_out), float("nan"), device="cuda", dtype=dtype)
        essa.essa_svdlora_forward(ctx, gp, X[:900], rd[:900], sAd, sBd, Y, flags | more)
        assert torch.equal(Y, got[0][0][:900])
        ref = orc.svdlora_forward(W, f, xv[:Rs[0]], r2c[:Rs[0]], sA, sB, base_only=more != 0)
        if dtype == torch.float32:
            assert orc.rel_errors(got[0][0].cpu().numpy(), ref)[1] <= EXACT_RMS
    gp.close()
    ctx.close()


@pytest.mark.parametrize("d_in,first", [(2048, 512), (3072, 385), (6144, 385), (6160, 512)])
def test_where_exact_products_begin(essa, d_in, first):
    """The line depends on rows and columns alone: exact products from it on, the fixed point's 3e-5 below it."""
    ctx = essa.Context(0)
    K, d_out, r = 3, 136, 8
    p = wl.make_projection("t", d_in, d_out, r, "int8", layer=19, proj=1)
    W, f = oracle_proj(p)
    gp = gpu_proj(essa, ctx, p)
    sA, sB = candidate_sigmas(f, K, 0.05)
    xb, xv = wl.make_x_bf16(first, d_in, x_id=65)
    r2c = np.random.default_rng(6).integers(0, K, first).astype(np.int32)
    X, rd, sAd, sBd, ref = bf16_dev(xb), to_dev(r2c), to_dev(sA), to_dev(sB), orc.svdlora_forward(W, f, xv, r2c, sA, sB)
    rms = []
    for R in (first - 1, first):
        Y = torch.empty(R, d_out, device="cuda")
        essa.essa_svdlora_forward(ctx, gp, X[:R], rd[:R], sAd, sBd, Y)
        rms.append(orc.rel_errors(Y.cpu().numpy(), ref[:R])[1])
    assert rms[1] <= 2e-6 < 1e-5 <= rms[0] <= 2e-4, rms     # 2^-24 sqrt(d_in / 32) and the 2^-17 of the rank-r term; half a unit of 16 bits
    gp.close()
    ctx.close()


@pytest.mark.parametrize("R,d_in,d_out,r", [
    (3, 400, 150, 8),              # fewer than eight K steps: one K part
    (3, 400, 150, 24),
    (130, 2064, 300, 16),          # eight K parts, the last step not full; a row block of two rows
    (130, 2064, 300, 32),
    (40, 8208, 64, 8),             # wider than the limb kernels go
])
def test_rank_term_of_the_exact_mode(essa, R, d_in, d_out, r):
    """The rank-r term alone, from the kernels of the exact product, with every bit of V_A's fp32 values.

    Rows (nearly) orthogonal to the columns of V_A: rounded to bf16 (2^-9 / sqrt(3) rms) they keep about 2^-10 of the t = V_A^T x
    that a row of that length would have, so an error of V_A shows 2^10 times as large as in an ordinary row.  fp32 V_A leaves
    2^-25 2^10 = 3e-5, the fp32 sums over the K steps as much again or twice, the bf16 head + tail of u and U_B 2^-17: 2e-4 is a bound.
    V_A as bf16 head + tail (2^-18) would leave 2e-3."""
    ctx = essa.Context(0)
    K = 3
    p = wl.make_projection("t", d_in, d_out, r, "int8", layer=15, proj=1)
    W, f = oracle_proj(p)
    gp = gpu_proj(essa, ctx, p)
    sA, sB = candidate_sigmas(f, K, 0.05)
    x = wl.make_x_bf16(R, d_in, x_id=61)[1].astype(np.float64)
    x -= (x @ f["V_A"]) @ f["V_A"].T
    X = torch.from_numpy(x).to(torch.bfloat16).cuda()
    r2c = np.random.default_rng(6).integers(0, K, R).astype(np.int32)
    ref = orc.svdlora_forward(np.zeros_like(W), f, X.double().cpu().numpy(), r2c, sA, sB)
    Y = torch.full((R, d_out), float("nan"), device="cuda")
    essa.essa_svdlora_forward(ctx, gp, X, to_dev(r2c), to_dev(sA), to_dev(sB), Y, essa.COMPUTE_BF16 | essa.LORA_ONLY)
    e_max, e_rms = orc.rel_errors(Y.cpu().numpy(), ref)
    print("rank term: R=%d d_in=%d r=%d rms %.3g max %.3g" % (R, d_in, r, e_rms, e_max), flush=True)
    assert e_rms <= 2e-4
    gp.close()
    ctx.close()


def test_rows_at_the_ends_of_the_range(essa):
    """Rows of 2^-90, 2^100 and 2^120 whose outputs are ordinary finite numbers, and channel scales of 2^-95 and 2^90 beside the usual
    ones: unscaled sums (70 sqrt(d_in) 2^120) or U_B over the scale would leave fp32.  Every row is held to the bar by itself."""
    ctx = essa.Context(0)
    R, d_in, d_out, r, K = 520, 1040, 300, 8, 3
    p = wl.make_projection("t", d_in, d_out, r, "int8", layer=16, proj=1)
    W, f = oracle_proj(p)
    sA, sB = candidate_sigmas(f, K, 0.05)
    xv = wl.make_x_bf16(R, d_in, x_id=62)[1].astype(np.float64)
    power = np.array([0, -90, 100, 120])[np.arange(R) % 4]
    X = torch.from_numpy(np.ldexp(xv, power[:, None])).to(torch.bfloat16).cuda()
    r2c = np.random.default_rng(6).integers(0, K, R).astype(np.int32)
    rd, sAd, sBd = to_dev(r2c), to_dev(sA), to_dev(sB)
    ref = orc.svdlora_forward(W, f, X.double().cpu().numpy(), r2c, sA, sB)
    gp = gpu_proj(essa, ctx, p)
    for flags in (0, essa.COMPUTE_BF16):
        Y = torch.empty(R, d_out, device="cuda")
        essa.essa_svdlora_forward(ctx, gp, X, rd, sAd, sBd, Y, flags)
        err = np.linalg.norm(Y.double().cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert np.all(err <= EXACT_RMS), (flags, err.max())
    gp.close()
    p.scales[7], p.scales[8] = 2.0 ** -95, -(2.0 ** 90)     # ordinary rows against extreme channels
    W, f = oracle_proj(p)
    gp = gpu_proj(essa, ctx, p)
    rows = power == 0
    Xs, refs = X[torch.from_numpy(rows).cuda()].repeat(4, 1).contiguous(), np.tile(orc.svdlora_forward(W, f, X.double().cpu().numpy()[rows], r2c[rows], sA, sB), (4, 1))
    Y = torch.empty(R, d_out, device="cuda")
    essa.essa_svdlora_forward(ctx, gp, Xs, to_dev(np.tile(r2c[rows], 4)), sAd, sBd, Y, 0)
    got = Y.double().cpu().numpy()
    for cols in (slice(7, 8), slice(8, 9), np.r_[0:7, 9:d_out]):
        assert np.linalg.norm(got[:, cols] - refs[:, cols]) <= EXACT_RMS * np.linalg.norm(refs[:, cols])
    gp.close()
    ctx.close()


def test_what_the_exact_product_cannot_take(essa):
    """A channel scale below its range keeps a projection on the fixed-point kernels at every row count, here on the 128 x 256 tile:
    two limbs, ragged rows and channels, both output types, the reward partials."""
    ctx = essa.Context(0)
    R, d_in, d_out, r, K = 2050, 192, 15400, 16, 3
    p = wl.make_projection("t", d_in, d_out, r, "int8", layer=17, proj=1)
    p.scales[5] = 1e-36
    W, f = oracle_proj(p)
    gp = gpu_proj(essa, ctx, p)
    sA, sB = candidate_sigmas(f, K, 0.05)
    xb, xv = wl.make_x_bf16(R, d_in, x_id=63)
    r2c = np.random.default_rng(6).integers(0, K, R).astype(np.int32)
    Xd, rd, sAd, sBd = bf16_dev(xb), to_dev(r2c), to_dev(sA), to_dev(sB)
    Y = torch.empty(R, d_out, device="cuda")
    essa.essa_svdlora_forward(ctx, gp, Xd, rd, sAd, sBd, Y)
    ref = orc.svdlora_forward(W, f, xv, r2c, sA, sB)
    assert orc.rel_errors(Y.cpu().numpy(), ref)[1] <= 2e-4      # the repository's bar for the fixed point
    assert np.abs(Y[:, 5].double().cpu().numpy() - ref[:, 5]).max() <= 2e-3 * np.abs(ref).max()      # the rank-r term alone in that channel
    Yb, v = torch.empty(R, d_out, device="cuda", dtype=torch.bfloat16), torch.randn(d_out, device="cuda")
    nblk = (d_out + 127) // 128
    rowpart = torch.full((nblk, R), float("nan"), device="cuda")
    essa.essa_svdlora_forward_reward_group(ctx, [(gp, Xd, rd, sAd, sBd, Yb)], [v], rowpart, 0)
    assert torch.equal(Yb, Y.to(torch.bfloat16))
    pad = torch.zeros(R, nblk * 128 - d_out, device="cuda", dtype=torch.float64)
    want = torch.cat([Yb.double() * v.double(), pad], 1).view(R, nblk, 128)
    assert torch.all((rowpart.T.double() - want.sum(2)).abs() <= 128 * 2.0 ** -24 * want.abs().sum(2) + 1e-30)
    gp.close()
    ctx.close()


def test_copy_of_the_weights_leaves_half_of_the_card(essa):
    """A projection created while less than half of the card is free takes no bf16 copy (2 bytes a weight on top of 2) and works all
    the same: the fixed point's error by itself, exact products by the flag."""
    ctx = essa.Context(0)
    R, d_in, d_out, r, K = 520, 4096, 4096, 8, 3
    p = wl.make_projection("t", d_in, d_out, r, "int8", layer=20, proj=1)
    W, f = oracle_proj(p)
    sA, sB = candidate_sigmas(f, K, 0.05)
    xb, xv = wl.make_x_bf16(R, d_in, x_id=66)
    r2c = np.random.default_rng(6).integers(0, K, R).astype(np.int32)
    X, rd, sAd, sBd = bf16_dev(xb), to_dev(r2c), to_dev(sA), to_dev(sB)
    Y = torch.empty(R, d_out, device="cuda")
    sample = np.arange(0, R, 37)
    ref = orc.svdlora_forward(W, f, xv[sample], r2c[sample], sA, sB)

    def error(gp, flags):
        essa.essa_svdlora_forward(ctx, gp, X, rd, sAd, sBd, Y, flags)
        return orc.rel_errors(Y.cpu().numpy()[sample], ref)[1]

    def create():
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        gp = gpu_proj(essa, ctx, p)
        return gp, before - torch.cuda.mem_get_info()[0]

    roomy, taken = create()
    assert taken >= 4 * d_in * d_out and error(roomy, 0) <= 2e-6
    free, total = torch.cuda.mem_get_info()
    fill = [torch.empty(free - total // 2, dtype=torch.uint8, device="cuda")]
    while torch.cuda.mem_get_info()[0] >= total // 2:
        fill.append(torch.empty(64 << 20, dtype=torch.uint8, device="cuda"))
    try:
        tight, taken = create()
    finally:
        del fill
        torch.cuda.empty_cache()
    assert 2 * d_in * d_out <= taken < 3 * d_in * d_out
    assert 1e-5 <= error(tight, 0) <= 2e-4                  # the repository's bar for the fixed point
    assert error(tight, essa.COMPUTE_BF16) <= EXACT_RMS
    assert error(roomy, 0) <= 2e-6                          # a copy that is there stays
    tight.close()
    roomy.close()
    ctx.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_tile_heights(essa, dtype):
    """Every tile that a row count can be given: at 1040 -> 4200 these take, in turn, 128 x 128 tiles with five stages, 160 x 128, 128 x 128
    twice a CU, 160 x 256, 192 x 256, 224 x 256 and 256 x 256.  The rows repeat the first 600, so each has the bits of the row that it
    repeats wherever it falls in its tile; those meet the oracle."""
    ctx = essa.Context(0)
    K, d_in, d_out, base = 4, 1040, 4200, 600
    p = wl.make_projection("t", d_in, d_out, 24, "int8", layer=19, proj=2)
    W, f = oracle_proj(p)
    gp = gpu_proj(essa, ctx, p)
    sA, sB = candidate_sigmas(f, K, 0.05)
    xb, xv = wl.make_x_bf16(base, d_in, x_id=65)
    r2c = np.random.default_rng(9).integers(0, K, base).astype(np.int32)
    X, rd, sAd, sBd = bf16_dev(xb), to_dev(r2c), to_dev(sA), to_dev(sB)
    v = torch.randn(d_out, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    first = None
    for R in (base, 1000, 1187, 2050, 2500, 3000, 3840):
        print("R=%d" % R, flush=True)
        at = torch.arange(R, device="cuda") % base
        Y = torch.full((R, d_out), float("nan"), device="cuda", dtype=dtype)
        part = torch.full(((d_out + 127) // 128, R), float("nan"), device="cuda")
        essa.essa_svdlora_forward_reward_group(ctx, [(gp, X[at].contiguous(), rd[at].contiguous(), sAd, sBd, Y)], [v], part, 0)
        first = first or (Y, part)
        assert torch.equal(Y, first[0][at]) and torch.equal(part, first[1][:, at])
    ref = orc.svdlora_forward(W, f, xv, r2c, sA, sB)
    if dtype == torch.float32:
        assert orc.rel_errors(first[0].cpu().numpy(), ref)[1] <= EXACT_RMS
    else:
        assert orc.rel_errors(bf16_host(first[0]), orc.round_to_bf16(ref))[1] <= BF16_RMS
    gp.close()
    ctx.close()
