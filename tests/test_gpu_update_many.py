"""The sign-probe update for more than 16 probes of a large model (workgroups of
four tiles with replicated tables) against the oracle on sampled parameters:
tile edges, the last partial tile, group remainders of 1, 8, 9 and 16 probes,
the cached sign words, a non-finite loss; more than 512 probes, past which the
workgroups work out the coefficients again."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import oracle  # noqa: E402
from paper_2505_17852_amd import workloads as wl  # noqa: E402


@pytest.fixture(scope="module")
def zo():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_17852_amd import zo as z
    z.lib()
    return z


@pytest.mark.parametrize("wdtype", [wl.FP32, wl.BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("N", [17, 24, 41, 64])
def test_many_probes_large_model(zo, N, wdtype):
    # 17.6 M parameters: over 2,048 tiles of 8,192, not a whole number of them
    cfg = dict(n_layers=1, vocab=16411, embed=512, hidden=512, wdtype=wdtype, probe=wl.RADEMACHER)
    P = zo.param_count(cfg)
    assert P > 2048 * 8192 and P % 8 != 0
    print(f"update many N={N} wdtype={wdtype} P={P}", flush=True)
    theta = zo.new_theta(cfg)
    zo.init(cfg, theta, 3)
    before = theta.clone()
    rng = np.random.default_rng(N)
    lp = (9.7 + 1e-3 * rng.standard_normal(N)).astype(np.float32)
    lm = (9.7 + 1e-3 * rng.standard_normal(N)).astype(np.float32)
    eps, lr, seed, i0 = 1e-3, 1e-1, 77, 3
    d = [torch.from_numpy(x).cuda() for x in (lp, lm)]
    skipped = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    zo.update(cfg, theta, seed, eps, lr, *d, i0=i0, skipped=skipped)
    assert int(skipped) == 0
    edges = np.array([0, 8191, 8192, 4 * 8192 - 1, 4 * 8192, 512 * 8192, P - 9, P - 8, P - 2, P - 1])
    idx = np.unique(np.concatenate([edges, rng.integers(0, P, 3000)])).astype(np.uint64)
    # sum_n c_n z_n[j] in 64 bits, c_n as the update defines it (fp32 of a double)
    c = ((np.float64(np.float32(lr)) / N) * ((lp.astype(np.float64) - lm) / (2.0 * np.float64(np.float32(eps))))).astype(np.float32)
    z = np.stack([np.array([oracle.probe(wl.RADEMACHER, seed, i0 + n, int(j), 1)[0] for j in idx]) for n in range(N)])
    old = before[torch.from_numpy(idx.astype(np.int64)).cuda()].float().cpu().numpy().astype(np.float64)
    new = theta[torch.from_numpy(idx.astype(np.int64)).cuda()].float().cpu().numpy().astype(np.float64)
    want = old - (c.astype(np.float64)[:, None] * z).sum(0)
    # N fp32 additions of terms of at most sum |c|, then fp32's or bf16's rounding of the result
    tol = N * 2.0 ** -24 * np.abs(c).sum() + np.abs(want) * 2.0 ** (-23 if wdtype == wl.FP32 else -8)
    assert np.all(np.abs(new - want) <= tol)
    if wdtype == wl.BF16:
        ws = zo.new_workspace(cfg, N, 1, 1)
        tok = torch.zeros((1, 2), dtype=torch.int32, device="cuda")
        zo.perturbed_losses(cfg, before, seed, eps, N, tok, i0=i0, workspace=ws)
        other = before.clone()
        zo.update_cached(cfg, other, seed, eps, lr, *d, zo.probe_bits(cfg, N, 1, 1, ws), i0=i0)
        assert torch.equal(other, theta)
    d[0][N - 1] = float("inf")
    kept = theta.clone()
    zo.update(cfg, theta, seed, eps, lr, *d, i0=i0, skipped=skipped)
    assert int(skipped) == 1 and torch.equal(theta, kept)


@pytest.mark.parametrize("N", [512, 513, 1041])
def test_coefficients_past_512_probes(zo, N):
    """A workgroup of 512 threads holds 512 coefficients at a time. Probe values
    from the library's own stream (checked against the oracle elsewhere)."""
    cfg = dict(n_layers=1, vocab=16411, embed=512, hidden=512, wdtype=wl.FP32, probe=wl.RADEMACHER)
    P = zo.param_count(cfg)
    print(f"update many N={N} P={P}", flush=True)
    theta = zo.new_theta(cfg)
    zo.init(cfg, theta, 3)
    before = theta.clone()
    rng = np.random.default_rng(N)
    lp = (9.7 + 1e-3 * rng.standard_normal(N)).astype(np.float32)
    lm = (9.7 + 1e-3 * rng.standard_normal(N)).astype(np.float32)
    eps, lr, seed, i0 = 1e-3, 1e-1, 77, 3
    zo.update(cfg, theta, seed, eps, lr, *[torch.from_numpy(x).cuda() for x in (lp, lm)], i0=i0)
    c = ((np.float64(np.float32(lr)) / N) * ((lp.astype(np.float64) - lm) / (2.0 * np.float64(np.float32(eps))))).astype(np.float32)
    n = 4096
    for j in (0, 512 * 8192 - n // 2, P - n):
        want = before[j:j + n].double()
        for k in range(N):
            want -= float(c[k]) * zo.debug_probe(wl.RADEMACHER, seed, i0 + k, j, n).double()
        # N fp32 additions of terms of at most sum |c|, then fp32's rounding of the result
        tol = N * 2.0 ** -24 * float(np.abs(c).sum()) + want.abs() * 2.0 ** -23
        assert torch.all((theta[j:j + n].double() - want).abs() <= tol)
