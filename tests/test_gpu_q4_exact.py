"""GPU parity of the exact-product kernel for 4-bit weights (codes as bf16, fp32 group sums) at the edges of its tiles.

Products are exact, fp32 sums random-signed and the zero-point term's operands fp32 numbers in three bf16 parts: 2e-6 for zero-mean rows.  (With two
parts each was off by 2^-18 rms of a term 5.2 times the output's rms, 2.8e-5 together; the bar below still is that.)"""
import numpy as np
import pytest
import torch

import essa_workloads as wl
import oracle as orc
from helpers import bf16_dev, bf16_host, candidate_sigmas, gpu_proj, oracle_proj, to_dev

pytestmark = pytest.mark.gpu

Q4_RMS, Q4_MAX = 3e-5, 3e-4
BF16_RMS, BF16_MAX = 1e-3, 2e-2


@pytest.mark.parametrize("d_in,d_out,r,Rs", [
    (2048, 2100, 24, (750, 1029, 1360, 1805, 2000, 2260)),   # tiles of 32, 48, 48 and 64 x 128, 80 and 96 x 256; output width not a multiple of 8
    (1152, 1400, 16, (1100, 1110, 2030, 2300, 3001, 3400, 4470)),   # nine groups: 48, 32, 48 and 64 x 128, 80, 96 and 64 x 256
    (4224, 264, 7, (513, 777)),                           # 33 groups: past one window of group sums, the last K part alone in the next
])
def test_q4_exact_tiles(essa, d_in, d_out, r, Rs):
    """The rows repeat the first `base`, so each has the bits of the row that it repeats wherever it falls in whatever tile (at row counts
    for which the rank-r term's K is cut alike)."""
    ctx = essa.Context(0)
    K, base = 4, 500
    p = wl.make_projection("t", d_in, d_out, r, "int4", layer=21, proj=1)
    W, f = oracle_proj(p)
    gp = gpu_proj(essa, ctx, p)
    sA, sB = candidate_sigmas(f, K, 0.05)
    xb, xv = wl.make_x_bf16(base, d_in, x_id=71)
    # rows at the ends of the format: nothing in between overflows or vanishes
    big, small = np.float32(2.0) ** 114, np.float32(2.0) ** -90
    xv = xv.copy()
    xv[7] *= big
    xv[8] *= small
    X = torch.from_numpy(xv).cuda().bfloat16()
    r2c = np.random.default_rng(9).integers(0, K, base).astype(np.int32)
    rd, sAd, sBd = to_dev(r2c), to_dev(sA), to_dev(sB)
    ref = orc.svdlora_forward(W, f, xv, r2c, sA, sB)
    unit = np.ones((base, 1))
    unit[7], unit[8] = 1.0 / float(big), 1.0 / float(small)
    nblk = (d_out + 127) // 128
    v = torch.randn(d_out, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    for dtype in (torch.float32, torch.bfloat16):
        first = None
        for R in Rs:
            print("q4 exact: d_in=%d d_out=%d r=%d R=%d %s" % (d_in, d_out, r, R, dtype), flush=True)
            at = torch.arange(R, device="cuda") % base
            Y = torch.full((R, d_out), float("nan"), device="cuda", dtype=dtype)
            part = torch.full((nblk, R), float("nan"), device="cuda")
            essa.essa_svdlora_forward_reward_group(ctx, [(gp, X[at].contiguous(), rd[at].contiguous(), sAd, sBd, Y)], [v], part, 0)
            first = first or (Y[:base], part[:, :base])
            assert torch.equal(Y, first[0][at]) and torch.equal(part, first[1][:, at])
        got = (first[0].cpu().numpy() if dtype == torch.float32 else bf16_host(first[0])).astype(np.float64) * unit
        want = (ref if dtype == torch.float32 else orc.round_to_bf16(ref)) * unit
        e_max, e_rms = orc.rel_errors(got, want)
        assert (e_rms <= Q4_RMS and e_max <= Q4_MAX) if dtype == torch.float32 else (e_rms <= BF16_RMS and e_max <= BF16_MAX), (e_rms, e_max)
        for i in (7, 8):
            assert orc.rel_errors(got[i], want[i])[1] <= (2 * Q4_RMS if dtype == torch.float32 else 3 * BF16_RMS)
        # the partials are sums of 128 products of the outputs as written, in fp32
        pad = torch.zeros(base, nblk * 128 - d_out, device="cuda", dtype=torch.float64)
        parts = torch.cat([first[0].double() * v.double(), pad], 1).view(base, nblk, 128)
        assert torch.all((first[1].T.double() - parts.sum(2)).abs() <= 128 * 2.0 ** -24 * parts.abs().sum(2) + 1e-30)
    # a non-finite entry spoils its own row and nothing else
    R = Rs[0]
    at = torch.arange(R, device="cuda") % base
    Xb = X[at].contiguous()
    for bad in (float("inf"), float("nan")):
        Xb[R - 2, d_in - 1] = bad
        Y = torch.empty(R, d_out, device="cuda")
        essa.essa_svdlora_forward(ctx, gp, Xb, rd[at].contiguous(), sAd, sBd, Y)
        Y0 = torch.empty(R, d_out, device="cuda")
        essa.essa_svdlora_forward(ctx, gp, X[at].contiguous(), rd[at].contiguous(), sAd, sBd, Y0)
        keep = torch.arange(R, device="cuda") != R - 2
        assert torch.isnan(Y[R - 2]).all() and torch.equal(Y[keep], Y0[keep])
    gp.close()
    ctx.close()


def test_q4_exact_group_and_limbs(essa):
    """A group on two inputs, ranks 16 and 32 mixed: the bits of single calls, whichever tile each gets; and next to the limb path, which
    takes the same rows when there are fewer of them, within both paths' noise (2^-16 of the row's largest entry, 3.5e-5 here)."""
    ctx = essa.Context(0)
    R, K, d_in = 700, 5, 3072
    specs = [(3072, 16), (520, 32), (40, 7), (1000, 24)]
    Xs = [bf16_dev(wl.make_x_bf16(R, d_in, x_id=80 + i)[0]) for i in range(2)]
    rd = to_dev(np.random.default_rng(8).integers(0, K, R).astype(np.int32))
    items = []
    for i, (d_out, r) in enumerate(specs):
        p = wl.make_projection("t", d_in, d_out, r, "int4", layer=22, proj=i)
        _, f = oracle_proj(p)
        sA, sB = candidate_sigmas(f, K, 0.05, i)
        items.append([gpu_proj(essa, ctx, p), Xs[i == 3], rd, to_dev(sA), to_dev(sB), torch.empty(R, d_out, device="cuda")])
    essa.essa_svdlora_forward_group(ctx, [tuple(it) for it in items])
    for it in items:
        print("d_out=%d" % it[0].d_out, flush=True)
        Y = torch.empty_like(it[5])
        essa.essa_svdlora_forward(ctx, *it[:5], Y)
        assert torch.equal(Y, it[5])
        few = torch.empty(256, it[0].d_out, device="cuda")
        essa.essa_svdlora_forward(ctx, it[0], it[1][:256].contiguous(), rd[:256].contiguous(), it[3], it[4], few)
        assert (few - Y[:256]).norm() <= 8e-5 * few.norm()
        it[0].close()
    ctx.close()


def test_q4_exact_rows_past_4_gib(essa):
    """An X of more than 4 GiB: the last tiles' rows are the rows that they repeat, as a small call has them (the rank-r term's K may be cut
    otherwise there: fp32 sums)."""
    ctx = essa.Context(0)
    d_in, d_out, r, K, base = 8192, 72, 8, 4, 701
    R = 2 ** 32 // (2 * d_in) + 131
    p = wl.make_projection("t", d_in, d_out, r, "int4", layer=23, proj=0)
    _, f = oracle_proj(p)
    gp = gpu_proj(essa, ctx, p)
    sAd, sBd = (to_dev(s) for s in candidate_sigmas(f, K, 0.05))
    few = bf16_dev(wl.make_x_bf16(base, d_in, x_id=72)[0])
    r2c = to_dev(np.random.default_rng(10).integers(0, K, base).astype(np.int32))
    at = torch.arange(R, device="cuda") % base
    X, rd = few[at], r2c[at].contiguous()
    print("q4 exact: d_in=%d d_out=%d R=%d" % (d_in, d_out, R), flush=True)
    Y, Yf = torch.empty(R, d_out, device="cuda"), torch.empty(base, d_out, device="cuda")
    essa.essa_svdlora_forward(ctx, gp, X, rd, sAd, sBd, Y)
    essa.essa_svdlora_forward(ctx, gp, few, r2c, sAd, sBd, Yf)
    off = (Y - Yf[at]).norm(dim=1) / Yf[at].norm(dim=1)
    assert off.max().item() <= 1e-5, (off.max().item(), int(off.argmax()))
    gp.close()
    ctx.close()


@pytest.mark.parametrize("d_in", [1152, 3584, 8192])
def test_q4_exact_rows_with_a_mean(essa, d_in):
    """Rows whose entries have a mean: the zero-point term, out of three bf16 parts a side and so fp32, starts the totals at the sum of G group terms
    of rms t = 24 s X_g, and the groups' own sums bring them back one by one.  Each of these additions is off by at most 2^-24 of what is
    left: root of their squares 2^-24 t sqrt(sum k^2) = 2^-24 t G^1.5 / sqrt(3).  The rank-r term has three operands in bf16 head and tail (V_A, u,
    U_B), each off by 2^-17 at most: sqrt(3) 2^-18 of its rms.  And no less exact than the fixed-point path."""
    ctx = essa.Context(0)
    d_out, r, K, R = 328, 16, 3, 1100
    p = wl.make_projection("t", d_in, d_out, r, "int4", layer=24, proj=2)
    W, f = oracle_proj(p)
    gp = gpu_proj(essa, ctx, p)
    sA, sB = candidate_sigmas(f, K, 0.05)
    g = torch.Generator(device="cuda").manual_seed(d_in)
    N = torch.randn(R, d_in, device="cuda", generator=g)
    r2c = (np.arange(R) % K).astype(np.int32)
    for name, X in (("N", N), ("|N|", N.abs()), ("1 + N", 1 + N), ("1 + 0.1 N", 1 + 0.1 * N), ("-3 + N", N - 3)):
        X = X.bfloat16()
        err = []
        xv = X[:200].double().cpu().numpy()
        ref = orc.svdlora_forward(W, f, xv, r2c[:200], sA, sB)
        for rows in (R, 200):                              # exact products, fixed point
            Y = torch.empty(rows, d_out, device="cuda")
            essa.essa_svdlora_forward(ctx, gp, X[:rows].contiguous(), to_dev(r2c[:rows]), to_dev(sA), to_dev(sB), Y)
            err.append(orc.rel_errors(Y[:200].cpu().numpy().astype(np.float64), ref)[1])
        scales = np.asarray(p.scales, np.float64)
        sums, rank = xv.reshape(200, -1, 128).sum(2), ref - xv @ np.asarray(W, np.float64).T
        t = 24.0 * np.sqrt((sums ** 2).mean() * (scales ** 2).mean())
        fold = 2.0 ** -24 * t * (d_in / 128) ** 1.5 / np.sqrt(3.0)
        bar = (fold + np.sqrt(3.0) * 2.0 ** -18 * np.sqrt((rank ** 2).mean())) / np.sqrt((ref ** 2).mean())
        print("d_in=%d x=%s exact %.2e fixed point %.2e bar %.2e" % (d_in, name, err[0], err[1], bar), flush=True)
        assert err[0] <= bar and err[0] <= err[1], (name, err, bar)
    gp.close()
    ctx.close()


def test_q4_copy_leaves_half_of_the_card(essa):
    """A 4-bit projection created while less than half of the card is free takes neither the copy of its codes (half a byte a weight) nor the operand that
    goes with it, and works all the same, with the fixed point's error."""
    ctx = essa.Context(0)
    R, d_in, d_out, r, K = 600, 4096, 4096, 8, 3
    p = wl.make_projection("t", d_in, d_out, r, "int4", layer=26, proj=1)
    W, f = oracle_proj(p)
    sA, sB = candidate_sigmas(f, K, 0.05)
    xb, xv = wl.make_x_bf16(R, d_in, x_id=73)
    r2c = np.random.default_rng(6).integers(0, K, R).astype(np.int32)
    X, rd, sAd, sBd = bf16_dev(xb), to_dev(r2c), to_dev(sA), to_dev(sB)
    Y = torch.empty(R, d_out, device="cuda")
    sample = np.arange(0, R, 37)
    ref = orc.svdlora_forward(W, f, xv[sample], r2c[sample], sA, sB)

    def error(gp):
        essa.essa_svdlora_forward(ctx, gp, X, rd, sAd, sBd, Y)
        return orc.rel_errors(Y.cpu().numpy()[sample], ref)[1]

    def create():
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        gp = gpu_proj(essa, ctx, p)
        return gp, before - torch.cuda.mem_get_info()[0]

    roomy, with_copy = create()
    assert error(roomy) <= Q4_RMS
    free, total = torch.cuda.mem_get_info()
    fill = [torch.empty(free - total // 2, dtype=torch.uint8, device="cuda")]
    while torch.cuda.mem_get_info()[0] >= total // 2:
        fill.append(torch.empty(64 << 20, dtype=torch.uint8, device="cuda"))
    try:
        tight, without = create()
    finally:
        del fill
        torch.cuda.empty_cache()
    assert with_copy - without >= d_in * d_out // 2
    assert 1e-5 <= error(tight) <= 2e-4                     # the repository's bar for the fixed point
    assert error(roomy) <= Q4_RMS                           # a copy that is there stays
    tight.close()
    roomy.close()
    ctx.close()
