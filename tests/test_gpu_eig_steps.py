"""The eigendecomposition's correction steps: where they take over from the sweeps and where they must not."""
import contextlib
import io
import os
import subprocess
import sys
import textwrap

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def essa():
    import paper_2507_04453_amd as m
    return m


def _check(st, C):
    """The defining identities; C is fp32 and B, D are rounded to fp32, so 2e-6 relative as for a cold start."""
    n = C.shape[0]
    B, D = st["B"].astype(np.float64), st["D"].astype(np.float64)
    lam = np.linalg.eigvalsh((C.astype(np.float64) + C.T) / 2)
    np.testing.assert_allclose(np.sort(D), np.sqrt(np.maximum(lam, 0)), rtol=2e-6, atol=1e-7 * np.sqrt(lam.max()))
    assert np.abs((B * D ** 2) @ B.T - C).max() <= 2e-6 * np.abs(C).max()
    assert np.abs(B.T @ B - np.eye(n)).max() <= 2e-6


def _load(cma, essa, C):
    n = C.shape[0]
    z = np.zeros(n, np.float32)
    cma.import_blob(essa.CmaState.pack_blob(n, 3, 0.5, z, z, z, np.ones(n, np.float32), C, np.eye(n, dtype=np.float32)))


# sizes around the 64-wide tiles; eps: how far C is from diagonal against a spacing of about 2 % between eigenvalues --
# from nothing to do, over steps alone, to steps that are refused (row sums of the corrections above 1/2)
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 130, 200])
@pytest.mark.parametrize("eps", [0.0, 1e-9, 1e-5, 1e-3, 0.3])
def test_near_diagonal(essa, n, eps):
    print("n=%d eps=%g" % (n, eps), flush=True)
    g = np.random.default_rng(1000 * n + int(eps * 1e6))
    d = 0.25 * 1.02 ** g.permutation(n)
    N = g.standard_normal((n, n)) / np.sqrt(n)
    C = (np.diag(d) + eps * np.sqrt(np.outer(d, d)) * (N + N.T) / 4).astype(np.float32)
    C = ((C + C.T) / 2).astype(np.float32)
    ctx = essa.Context(0)
    cma = essa.CmaState(ctx, n, 0.32, None)
    _load(cma, essa, C)
    sweeps, off = cma.refresh_basis(ctx)
    assert off <= 1e-7
    first = cma.export()
    _check(first, C)
    assert cma.refresh_basis(ctx)[0] == 1                  # nothing left to do
    _check(cma.export(), C)
    cma.close()
    ctx.close()


# equal eigenvalues (one cluster, two clusters, pairs 1e-7 apart) and ones far below the largest: the sweeps' work
@pytest.mark.parametrize("kind", ["identity", "clusters", "close", "tiny", "indefinite"])
@pytest.mark.parametrize("n", [66, 128])
def test_spectra_that_steps_cannot_separate(essa, kind, n):
    print("n=%d %s" % (n, kind), flush=True)
    g = np.random.default_rng(n)
    Q = np.linalg.qr(g.standard_normal((n, n)))[0]
    lam = {"identity": np.ones(n), "clusters": np.where(np.arange(n) < n // 2, 1.0, 2.0), "close": 1.0 + np.arange(n) // 2 + 1e-7 * np.arange(n),
           "tiny": np.concatenate([np.full(n // 2, 1e-9), np.linspace(1, 2, n - n // 2)]), "indefinite": np.linspace(-1e-3, 1.0, n)}[kind]
    C = ((Q * lam) @ Q.T).astype(np.float32)
    C = ((C + C.T) / 2).astype(np.float32)
    ctx = essa.Context(0)
    cma = essa.CmaState(ctx, n, 0.32, None)
    _load(cma, essa, C)
    assert cma.refresh_basis(ctx)[1] <= 1e-7
    st = cma.export()
    if kind in ("tiny", "indefinite"):                     # D is clamped at zero there
        B = st["B"].astype(np.float64)
        assert np.abs(B.T @ B - np.eye(n)).max() <= 2e-6
        assert np.abs((B * st["D"].astype(np.float64) ** 2) @ B.T - C).max() <= max(2e-6, 1.1 * max(0.0, -lam.min())) * np.abs(C).max() * 2
    else:
        _check(st, C)
    cma.refresh_basis(ctx)
    cma.close()
    ctx.close()


@pytest.mark.parametrize("n,K,gens", [(130, 64, 12), (200, 24, 2)])
def test_refresh_after_generations(essa, n, K, gens):
    """Generations of update between refreshes: the basis follows C, columns keep their places and signs."""
    ctx = essa.Context(0)
    cma = essa.CmaState(ctx, n, 0.3, None)
    g = np.random.default_rng(n)
    C = np.diag(0.25 * 1.02 ** g.permutation(n)).astype(np.float32)
    _load(cma, essa, C)
    cma.refresh_basis(ctx)
    for rnd in range(3):
        before = cma.export()["B"].astype(np.float64)
        for _ in range(gens):
            seeds = torch.from_numpy(g.integers(-2 ** 31, 2 ** 31 - 1, K).astype(np.int32)).cuda()
            essa.essa_cmaes_update(ctx, cma, seeds, torch.from_numpy(g.standard_normal(K).astype(np.float32)).cuda(), None)
        print("n=%d round %d: %s" % (n, rnd, cma.refresh_basis(ctx)), flush=True)
        st = cma.export()
        _check(st, ((st["C"] + st["C"].T) / 2))
        assert np.median(np.sum(st["B"] * before, axis=0)) > 0.9
    cma.close()
    ctx.close()


def test_scratch_pinned_by_a_graph(essa):
    """With a recorded graph holding the scratch at its size, a refresh that fits only without the steps still runs."""
    n = 192
    side = torch.cuda.Stream()
    ctx = essa.Context(0, side)
    cma = essa.CmaState(ctx, n, 0.32, None)
    C = np.diag(np.linspace(1, 2, n)).astype(np.float32)
    C[0, 1] = C[1, 0] = 1e-4
    _load(cma, essa, C)
    # scratch by the sampler: 512 n floats, a quarter more and a megabyte = 1.54 MB; the sweeps alone need 1.48, with steps 1.88
    theta = torch.empty(512, n, device="cuda")
    seeds = torch.arange(512, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        essa.essa_sample_candidates(ctx, cma, seeds, theta)
        ctx.graph_begin()
        essa.essa_sample_candidates(ctx, cma, seeds, theta)
        graph = ctx.graph_end()
    cma.refresh_basis(ctx)
    _check(cma.export(), C)
    graph.close()
    cma.refresh_basis(ctx)
    _check(cma.export(), C)
    cma.close()
    ctx.close()


def test_card_too_full_for_the_steps(essa):
    """A card with room for the sweeps' scratch but not for the steps' as well: the refresh does its work on the sweeps."""
    n = 8192
    ctx = essa.Context(0)
    warm = essa.CmaState(ctx, 64, 0.32, None)
    warm.refresh_basis(ctx)                                # the kernels are loaded before the card fills up
    cma = essa.CmaState(ctx, n, 0.32, None)
    d = np.linspace(1, 2, n).astype(np.float32)
    zero = np.zeros(n, np.float32)
    cma.import_blob(essa.CmaState.pack_blob(n, 3, 0.5, zero, zero, zero, np.ones(n, np.float32), np.diag(d), np.eye(n, dtype=np.float32)))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    # the refresh wants scratch (a quarter more than it uses) and the fp64 basis: 1391 + 537 MB with the sweeps alone, 2098 + 537 MB
    # with the steps; the card is filled until 2098 MB can no longer be had at once and the first two still can
    def fits(*mb):
        try:
            held = [torch.empty(m * 10 ** 6, dtype=torch.uint8, device="cuda") for m in mb]
        except torch.OutOfMemoryError:
            held = None
        ok = held is not None
        del held
        torch.cuda.empty_cache()
        return ok

    fill = [torch.empty(torch.cuda.mem_get_info()[0] - 5 * 10 ** 9, dtype=torch.uint8, device="cuda")]
    try:
        while fits(2099):
            fill.append(torch.empty(48 << 20, dtype=torch.uint8, device="cuda"))
        assert fits(1392, 538), "no such filling found"
        print("card filled", flush=True)
        cma.refresh_basis(ctx)
    finally:
        del fill
        torch.cuda.empty_cache()
    st = cma.export()
    assert np.array_equal(st["B"], np.eye(n, dtype=np.float32))
    np.testing.assert_allclose(st["D"], np.sqrt(d.astype(np.float64)), rtol=2e-7)
    warm.refresh_basis(ctx)                                # and no error is left behind for the next call
    cma.close()
    warm.close()
    ctx.close()


def _with_page_locked_memory_watched(tmp_path, body, refuse):
    """Runs `body` in a process of its own that counts the requests for 64 bytes of page-locked memory, or refuses them; what it printed, and the count."""
    (tmp_path / "watch.cpp").write_text(
        '#include <dlfcn.h>\n#include <cstddef>\nextern "C" {\nint asked = 0;\n'
        'int hipHostMalloc(void** p, size_t bytes, unsigned flags) {\n'
        '    if (bytes == 64 && (++asked, %d)) { *p = nullptr; return 2; }      // out of memory\n'
        '    static auto next = (int (*)(void**, size_t, unsigned))dlsym(dlopen("libamdhip64.so.7", RTLD_NOLOAD | RTLD_NOW), "hipHostMalloc");\n'
        '    return next(p, bytes, flags);\n}\n}\n' % refuse)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", str(tmp_path / "watch.cpp"), "-o", str(tmp_path / "watch.so"), "-ldl"], check=True)
    env = dict(os.environ, LD_PRELOAD=":".join(x for x in (str(tmp_path / "watch.so"), os.environ.get("LD_PRELOAD", "")) if x))
    code = "import ctypes, sys\nsys.path[:0] = %r\n" % ([os.path.dirname(os.path.dirname(os.path.abspath(__file__))), os.path.dirname(os.path.abspath(__file__))],)
    code += textwrap.dedent(body) + "\nprint(ctypes.c_int.in_dll(ctypes.CDLL(None), 'asked').value, flush=True)\n"
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = r.stdout.splitlines()
    return lines[:-1], int(lines[-1])


def test_refresh_without_page_locked_memory(essa, tmp_path):
    """The steps' numbers are then copied back: the same bits, steps and sweeps as with it, also for a second state of the context."""
    body = """
        import numpy as np, torch, hashlib
        import paper_2507_04453_amd as essa
        import test_gpu_eig_steps as t
        ctx = essa.Context(0)
        for n, seed in ((65, 1), (130, 2)):
            g = np.random.default_rng(seed)
            d = 0.25 * 1.02 ** g.permutation(n)
            cma = essa.CmaState(ctx, n, 0.32, None)
            for eps in (1e-3, 2e-3, 0.3):
                N = g.standard_normal((n, n)) / np.sqrt(n)
                C = (np.diag(d) + eps * np.sqrt(np.outer(d, d)) * (N + N.T) / 4).astype(np.float32)
                C = ((C + C.T) / 2).astype(np.float32)
                t._load(cma, essa, C)
                for again in range(2):
                    print(n, eps, cma.refresh_basis(ctx), hashlib.sha256(cma.export_blob()).hexdigest())
                t._check(cma.export(), C)
            cma.close()
        ctx.close()
    """
    without, refused = _with_page_locked_memory_watched(tmp_path, body, True)
    assert refused >= 1
    out = io.StringIO()
    with contextlib.redirect_stdout(out):
        exec(textwrap.dedent(body), {})
    assert without == out.getvalue().splitlines()


def test_page_locked_memory_is_asked_for_once_a_context(essa, tmp_path):
    """It takes as long as a small state's refresh: the states of a context share it."""
    body = """
        import paper_2507_04453_amd as essa
        ctx = essa.Context(0)
        for n in (8, 8, 65):
            cma = essa.CmaState(ctx, n, 0.32, None)
            cma.refresh_basis(ctx)
            cma.refresh_basis(ctx)
            cma.close()
        ctx.close()
    """
    assert _with_page_locked_memory_watched(tmp_path, body, False)[1] == 1
