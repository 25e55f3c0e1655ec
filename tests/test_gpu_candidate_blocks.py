"""The product of the normals with the basis takes its columns in passes of up to four blocks of 16: at every number of blocks, full
and ragged, a candidate has the bits that it has on its own (each output is one fixed-order sum), and the right value."""
import numpy as np
import pytest
import torch

from helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16, 67, 260])
def test_candidates_do_not_depend_on_their_number(essa, n):
    ctx = essa.Context(0)
    g = np.random.default_rng(n)
    Q = np.linalg.qr(g.standard_normal((n, n)))[0].astype(np.float32)
    d = np.exp(g.uniform(-0.7, 0.7, n)).astype(np.float32)
    cma = essa.CmaState(ctx, n, 0.32, g.standard_normal(n).astype(np.float32))
    cma.set_basis(to_dev(Q), to_dev(d))
    seeds = torch.arange(1, 146, dtype=torch.int32, device="cuda")
    one = torch.empty(145, n, device="cuda")
    for k in range(145):
        essa.essa_sample_candidates(ctx, cma, seeds[k:k + 1], one[k:k + 1])
    for K in (16, 17, 32, 33, 48, 49, 64, 65, 81, 96, 97, 128, 129, 144, 145):
        theta, z = torch.full((K, n), float("nan"), device="cuda"), torch.empty(K, n, device="cuda")
        essa.essa_sample_candidates(ctx, cma, seeds[:K], theta, z)
        assert torch.equal(theta, one[:K]), K
    want = cma.export()["m"].astype(np.float64) + np.float64(np.float32(0.32)) * (z.cpu().numpy().astype(np.float64) * d) @ Q.T.astype(np.float64)
    assert np.linalg.norm(theta.cpu().numpy() - want) <= 1e-6 * np.linalg.norm(want)      # fp32 sums over n
    cma.close()
    ctx.close()


def test_candidates_past_a_descriptor(essa):
    """More right-hand sides than a buffer descriptor's 2 GB: the last candidates are what they are on their own."""
    ctx = essa.Context(0)
    K, n = 32768 + 40, 16381
    print("K=%d n=%d" % (K, n), flush=True)
    cma = essa.CmaState(ctx, n, 0.32)
    seeds = torch.arange(1, K + 1, dtype=torch.int32, device="cuda")
    theta, few = torch.zeros(K, n, device="cuda"), torch.empty(4, n, device="cuda")
    essa.essa_sample_candidates(ctx, cma, seeds, theta)
    for k in (0, 16384, 32764, K - 4):
        essa.essa_sample_candidates(ctx, cma, seeds[k:k + 4].contiguous(), few)
        assert torch.equal(theta[k:k + 4], few) and few.abs().max().item() > 0, k
    cma.close()
    ctx.close()
