"""GPU parity of the fp32 product (fp32 activations, and bf16 rows that the matrix kernels do not take) at the edges of its tiles, K
steps and load forms.

Every product and sum is fp32: against the fp64 oracle the error of a sum of d_in products of random sign is about
2^-24 sqrt(d_in) of its size, the rank-r chain (three sums of at most d_in, r, r terms on a term a twentieth of the output) and the
scale add a few roundings more."""
import numpy as np
import pytest
import torch

import essa_workloads as wl
import oracle as orc
from helpers import bf16_dev, candidate_sigmas, gpu_proj, oracle_proj, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,d_in,d_out,r,quant,bf16,shift", [
    (3, 7, 9, 2, "int8", False, 0),          # less than one step, rows of no whole quads
    (17, 132, 33, 5, "int8", False, 0),      # second step of the first wave only, one row and one channel past a tile
    (16, 128, 16, 16, "int8", False, 1),     # exactly one tile; rows not aligned for 16-byte loads
    (70, 1030, 130, 16, "int8", False, 0),   # two trips, element by element
    (513, 516, 1040, 32, "int8", False, 0),  # 32 x 32 tiles
    (40, 256, 48, 4, "int4", False, 0),
    (20, 1152, 40, 8, "int4", False, 0),     # nine groups: the first wave takes two
    (520, 128, 1100, 8, "int4", False, 0),   # 4-bit weights on the 32 x 32 tiles
    (9, 256, 24, 8, "int4", False, 1),       # and with rows not aligned for 16-byte loads
    (21, 1152, 40, 8, "int4", False, 1),     # nine groups
    (33, 328, 96, 4, "int8", True, 0),       # bf16 rows of 8-byte multiples
    (33, 326, 96, 24, "int8", True, 0),      # bf16 rows of odd words
])
def test_f32_product(essa, R, d_in, d_out, r, quant, bf16, shift):
    ctx = essa.Context(0)
    K = 3
    print("f32 product: R=%d d_in=%d d_out=%d r=%d %s bf16=%s" % (R, d_in, d_out, r, quant, bf16), flush=True)
    p = wl.make_projection("t", d_in, d_out, r, quant, layer=12, proj=1)
    W, f = oracle_proj(p)
    gp = gpu_proj(essa, ctx, p)
    sA, sB = candidate_sigmas(f, K, 0.05)
    xb, xv = wl.make_x_bf16(R, d_in, x_id=33)
    if bf16:
        Xd = bf16_dev(xb)
    else:
        xv = xv + np.random.default_rng(2).standard_normal(xv.shape).astype(np.float32) * np.float32(1e-3)
        xv = xv.astype(np.float32)
        Xd = torch.empty(R * d_in + shift, device="cuda")[shift:].view(R, d_in)
        Xd.copy_(torch.from_numpy(xv))
    r2c = np.random.default_rng(6).integers(0, K, R).astype(np.int32)
    rd, sAd, sBd = to_dev(r2c), to_dev(sA), to_dev(sB)
    bar = 2.0 ** -24 * (np.sqrt(d_in) + 8)
    for flags, kw in ((0, {}), (essa.BASE_ONLY, {"base_only": True}), (essa.LORA_ONLY, {"lora_only": True})):
        Y = torch.full((R, d_out), float("nan"), device="cuda")
        essa.essa_svdlora_forward(ctx, gp, Xd, rd, sAd, sBd, Y, flags)
        e_max, e_rms = orc.rel_errors(Y.cpu().numpy(), orc.svdlora_forward(W, f, xv, r2c, sA, sB, **kw))
        assert e_rms <= (4 if flags == essa.LORA_ONLY else 1) * bar, (flags, e_rms, bar)   # the rank-r term alone: all of the chain's roundings
    good, bad = torch.empty(R, d_out, device="cuda"), torch.empty(R, d_out, device="cuda")
    essa.essa_svdlora_forward(ctx, gp, Xd, rd, sAd, sBd, good)
    Xbad = Xd.clone()
    Xbad[R // 2, d_in - 1] = float("inf")                  # a non-finite entry stays in its row
    essa.essa_svdlora_forward(ctx, gp, Xbad, rd, sAd, sBd, bad)
    keep = torch.arange(R, device="cuda") != R // 2
    assert not torch.isfinite(bad[R // 2]).any()
    # (with shift the clone is aligned and the rows themselves are not: the order of the sums does not hang on it)
    assert torch.equal(bad[keep], good[keep])
    gp.close()
    ctx.close()
