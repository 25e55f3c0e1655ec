"""int8 weights between the weight-streaming kernel and the exact product: 32- and 64-row tiles by what the busiest CU has to do."""
import numpy as np
import pytest
import torch

import oracle as orc

pytestmark = pytest.mark.gpu


# 12288 channels are 96 column tiles: a CU has at most one 64-row tile up to 128 rows, two up to 320, and of the 32-row tiles two up to 160, three up to 256, four up to
# 320, five from there on.  With two limbs 64-row tiles up to 128 rows, 32-row tiles from 129 to 256, then 64 again; with one limb 32-row tiles from 129 to 160 only.
# 321: both heights' last tiles have one row
@pytest.mark.parametrize("rows", [65, 97, 128, 129, 160, 161, 257, 321])
@pytest.mark.parametrize("mode", ["default", "w8a8"])
def test_rows_do_not_hang_on_their_tile(essa, mode, rows):
    d_in, d_out, r, K = 544, 12288 - 40, 8, 5
    g = np.random.default_rng(rows)
    ctx = essa.Context(0)
    W = g.integers(-127, 128, size=(d_out, d_in), dtype=np.int8)
    s = g.uniform(0.001, 0.01, d_out).astype(np.float32)
    proj = essa.Projection(ctx, W, s, None, (g.standard_normal((r, d_in)) / np.sqrt(d_in)).astype(np.float32), (0.1 * g.standard_normal((d_out, r))).astype(np.float32),
                           essa.QUANT_INT8_PERCH)
    sA, sB = (torch.from_numpy(g.standard_normal((K, r)).astype(np.float32)).cuda() for _ in range(2))
    X = torch.from_numpy(g.standard_normal((rows, d_in)).astype(np.float32)).cuda().bfloat16()
    r2c = torch.from_numpy(g.integers(0, K, rows).astype(np.int32)).cuda()
    flags = essa.COMPUTE_W8A8 if mode == "w8a8" else 0

    def call(lo, hi):
        Y = torch.full((hi - lo, d_out), float("nan"), device="cuda", dtype=torch.bfloat16)
        essa.essa_svdlora_forward_group(ctx, [(proj, X[lo:hi], r2c[lo:hi], sA, sB, Y)], flags)
        return Y

    whole = call(0, rows)
    parts = torch.cat([call(i, min(i + 32, rows)) for i in range(0, rows, 32)])          # the kernel without tiles
    torch.cuda.synchronize()
    assert torch.equal(whole.view(torch.int16), parts.view(torch.int16))
    # against fp32 sums of the same operands; the rank-r term is a few per cent of the output and left out of neither side by this bound:
    # without the base term the difference would be 1, and bf16 outputs of it round to 2^-9
    ref = X.float() @ (torch.from_numpy(W).cuda().float() * torch.from_numpy(s).cuda()[:, None]).T
    base = torch.full_like(whole, float("nan"))
    essa.essa_svdlora_forward_group(ctx, [(proj, X, r2c, sA, sB, base)], flags | essa.BASE_ONLY)
    torch.cuda.synchronize()
    # int8 codes of a row of N(0, 1): steps of amax / 127, about 3.3 / 127, uniform errors of 1 / sqrt(12) of one
    bound = 2 ** -8 if mode == "default" else 1.5 * 3.3 / 127 / np.sqrt(12)
    assert ((base.float() - ref).norm() / ref.norm()).item() <= bound
    proj.close()
    ctx.close()


@pytest.mark.parametrize("rows", [40, 65, 97, 128, 129, 160, 161])     # 32-row tiles at 40 and from 129 to 160
def test_int32_sums_of_both_heights(essa, rows):
    d_in, d_out = 544, 12288 - 40
    g = np.random.default_rng(rows)
    ctx = essa.Context(0)
    W = g.integers(-127, 128, size=(d_out, d_in), dtype=np.int8)
    proj = essa.Projection(ctx, W, np.ones(d_out, np.float32), None, (g.standard_normal((4, d_in)) / np.sqrt(d_in)).astype(np.float32),
                           g.standard_normal((d_out, 4)).astype(np.float32), essa.QUANT_INT8_PERCH)
    X = torch.from_numpy(g.standard_normal((rows, d_in)).astype(np.float32)).cuda().bfloat16()
    xq, xs = torch.empty(rows, d_in, dtype=torch.int8, device="cuda"), torch.empty(rows, device="cuda")
    acc = torch.full((rows, d_out), -2 ** 31, dtype=torch.int32, device="cuda")
    essa.essa_w8a8_accumulators(ctx, proj, X, xq, xs, acc)
    rq, rs = orc.quantize_rows_int8(X.float().cpu().numpy())
    assert np.array_equal(xq.cpu().numpy(), rq) and np.array_equal(xs.cpu().numpy(), rs)
    assert np.array_equal(acc.cpu().numpy(), (rq.astype(np.float64) @ W.T.astype(np.float64)).astype(np.int32))       # exact below 2^53
    proj.close()
    ctx.close()


# 5 and 2 column tiles: tiles that are no multiple of 8, fewer than 8, and as many as go evenly to the XCDs
@pytest.mark.parametrize("rows", [33, 65, 70, 129, 225, 256])
@pytest.mark.parametrize("quant,mode", [("int8", "default"), ("int8", "w8a8"), ("int4", "default")])
def test_uneven_numbers_of_tiles(essa, quant, mode, rows):
    d_in, r, K = 384, 8, 3
    g = np.random.default_rng(rows)
    ctx = essa.Context(0)
    flags = essa.COMPUTE_W8A8 if mode == "w8a8" else 0
    projs = []
    for d_out in (600, 200):
        A, B = (g.standard_normal((r, d_in)) / np.sqrt(d_in)).astype(np.float32), (0.1 * g.standard_normal((d_out, r))).astype(np.float32)
        if quant == "int8":
            projs.append(essa.Projection(ctx, g.integers(-127, 128, size=(d_out, d_in), dtype=np.int8), g.uniform(0.001, 0.01, d_out).astype(np.float32), None, A, B,
                                         essa.QUANT_INT8_PERCH))
        else:
            projs.append(essa.Projection(ctx, g.integers(0, 256, size=(d_out, d_in // 2), dtype=np.uint8), g.uniform(0.001, 0.01, (d_out, 3)).astype(np.float16),
                                         g.uniform(6.0, 9.0, (d_out, 3)).astype(np.float16), A, B, essa.QUANT_INT4_G128))
    sA, sB = (torch.from_numpy(g.standard_normal((K, r)).astype(np.float32)).cuda() for _ in range(2))
    X = torch.from_numpy(g.standard_normal((rows, d_in)).astype(np.float32)).cuda().bfloat16()
    r2c = torch.from_numpy(g.integers(0, K, rows).astype(np.int32)).cuda()

    def call(which):
        Y = [torch.full((rows, projs[i].d_out), float("nan"), device="cuda", dtype=torch.bfloat16) for i in which]
        essa.essa_svdlora_forward_group(ctx, [(projs[i], X, r2c, sA, sB, y) for i, y in zip(which, Y)], flags)
        torch.cuda.synchronize()
        return Y

    both = call((0, 1))
    assert all(torch.isfinite(y).all() for y in both)
    for i in (0, 1):                                       # the item alone: other tiles beside it, or none
        assert torch.equal(both[i].view(torch.int16), call((i,))[0].view(torch.int16))
    for p in projs:
        p.close()
    ctx.close()
