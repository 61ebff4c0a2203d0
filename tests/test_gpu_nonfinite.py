"""Non-finite logits: a NaN (fp32: or infinite) weight row of the head makes every
loss NaN also where it is alone in its vocabulary tile or wave, and a bias of
-inf takes its word out of the softmax and leaves the losses finite."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2505_17852_amd import workloads as wl  # noqa: E402


@pytest.fixture(scope="module")
def zo():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_17852_amd import zo as z
    z.lib()
    return z


# the last word alone in a tile of 128 (fp32) or 256 (bf16), or in a wave's 64 columns; not alone
@pytest.mark.parametrize("wdtype,V", [(wl.FP32, 129), (wl.FP32, 60), (wl.BF16, 257), (wl.BF16, 65), (wl.BF16, 60)])
def test_non_finite_logits(zo, oracle, wdtype, V):
    cfg = dict(n_layers=1, vocab=V, embed=64, hidden=64, wdtype=wdtype, probe=wl.RADEMACHER)
    print(f"non-finite {cfg}", flush=True)
    N, B, C, eps, H = 3, 5, 4, 1e-2, cfg["hidden"]
    tok = wl.uniform_tokens(np.random.default_rng(V), B, C, V - 1)  # the last word is never a target
    td = torch.from_numpy(tok).cuda()
    P = zo.param_count(cfg)

    def losses(poison):
        theta = zo.new_theta(cfg)
        zo.init(cfg, theta, 2)
        poison(theta)
        Lp, Lm = zo.perturbed_losses(cfg, theta, 8, eps, N, td)
        L, L0 = zo.fd_losses(cfg, theta, 8, eps, N, td)
        return torch.cat([Lp, Lm, L, L0])

    def row(value):
        return lambda theta: theta[P - V - H:P - V].fill_(value)

    for value in [float("nan")] + [float("inf")] * (wdtype == wl.FP32):
        assert torch.all(torch.isnan(losses(row(value)))), value
    got = losses(lambda theta: theta[P - 1:].fill_(float("-inf"))).cpu().numpy()
    ref = oracle.init(cfg, 2)
    # the oracle's bf16 parameters are their 16 bits
    ref[P - 1] = np.float32(-np.inf) if wdtype == wl.FP32 else np.uint16(0xFF80)
    rp, rm = oracle.perturbed_losses(cfg, ref, 8, eps, N, tok, as_double=True)
    rl, r0 = oracle.fd_losses(cfg, ref, 8, eps, N, tok)
    want = np.concatenate([rp, rm, rl, np.atleast_1d(r0)])
    assert np.all(np.abs(got - want) <= (1e-5 if wdtype == wl.FP32 else 2e-2) * want), (got, want)
