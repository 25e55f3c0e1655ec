"""GPU parity of the search's matrix kernels at dimensions that are not a multiple of 4 (rows that end inside a 16-byte load, rows
shorter than one): candidates and one update against fp64, bars as for other dimensions (fp32 sums over n)."""
import numpy as np
import pytest
import torch

from helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [5, 24, 70])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 6, 7, 17, 66, 131, 1795])
def test_odd_dimension(essa, n, K):
    ctx = essa.Context(0)
    g = np.random.default_rng(n)
    Q = np.linalg.qr(g.standard_normal((n, n)))[0].astype(np.float32)
    d = np.exp(g.uniform(-0.7, 0.7, n)).astype(np.float32)
    C0 = (Q.astype(np.float64) * d.astype(np.float64) ** 2) @ Q.T.astype(np.float64)
    C0 = ((C0 + C0.T) / 2).astype(np.float32)
    m0 = g.standard_normal(n).astype(np.float32)
    zero = np.zeros(n, np.float32)
    cma = essa.CmaState(ctx, n, 0.32, m0)
    cma.import_blob(essa.CmaState.pack_blob(n, 0, 0.32, m0, zero, zero, d, C0, Q))
    seeds = torch.arange(1, K + 1, dtype=torch.int32, device="cuda")
    theta, z = torch.empty(K, n, device="cuda"), torch.empty(K, n, device="cuda")
    essa.essa_sample_candidates(ctx, cma, seeds, theta, z)
    zz = z.cpu().numpy().astype(np.float64)
    y = (zz * d) @ Q.astype(np.float64).T
    want = m0 + np.float64(np.float32(0.32)) * y
    assert np.linalg.norm(theta.cpu().numpy() - want) <= 1e-6 * np.linalg.norm(want)
    F = g.standard_normal(K).astype(np.float32)
    essa.essa_cmaes_update(ctx, cma, seeds, to_dev(F))
    st = cma.export()
    order = np.argsort(-F, kind="stable")
    # the mean moves along the weighted best directions; C gains terms on exactly those and p_c, symmetrically
    mu = K // 2
    w = np.log((K + 1) / 2) - np.log(np.arange(1, mu + 1))
    w /= w.sum()
    want_m = m0 + np.float64(np.float32(0.32)) * (w @ y[order[:mu]])
    assert np.linalg.norm(st["m"] - want_m) <= 2e-6 * np.linalg.norm(want_m)
    assert np.array_equal(st["C"], st["C"].T)
    mu_eff = 1 / (w ** 2).sum()
    cc = (4 + mu_eff / n) / (n + 4 + 2 * mu_eff / n)
    c1 = 2 / ((n + 1.3) ** 2 + mu_eff)
    cmu = min(1 - c1, 2 * (mu_eff - 2 + 1 / mu_eff) / ((n + 2) ** 2 + mu_eff))
    pc = st["p_c"].astype(np.float64)
    hs = 1.0 if np.any(pc != 0) else 0.0
    want_C = (1 - c1 - cmu + (1 - hs) * c1 * cc * (2 - cc)) * C0 + c1 * np.outer(pc, pc) + cmu * (y[order[:mu]].T * w) @ y[order[:mu]]
    assert np.linalg.norm(st["C"] - want_C) <= 4e-6 * np.linalg.norm(want_C)
    cma.close()
    ctx.close()
