"""int8 weights between the weight-streaming kernel and the exact product: 32- and 64-row tiles by what the busiest CU has to do."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# 12288 channels are 96 column tiles: the 64-row tiles fill one round of CUs up to 128 rows, two from 129 on, the 32-row tiles two of their own up to
# 160, three up to 256, four up to 320: the rule changes its mind at 129, 161, 257 and 321, with two limbs and with one not at the same places
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
