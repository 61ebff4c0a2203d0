"""Batches of one position (C = 1) against the oracle, for models with several
column blocks per launch and launches of more workgroups than are resident at
once: every workgroup must read the zero state before the first timestep,
whatever the others have written by then. The workspace is filled with NaN
before the call."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2505_17852_amd import workloads as wl  # noqa: E402

# the bars of the two paths' other tests against the oracle (fp32 sums; fp16 operands)
RTOL = {wl.FP32: 1e-5, wl.BF16: 2e-2}


@pytest.fixture(scope="module")
def zo():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_17852_amd import zo as z
    z.lib()
    return z


# (L, E, H, N, B): the narrowest width with two column blocks for over 600 probes, wider ones
SHAPES = {wl.FP32: [(1, 32, 32, 601, 4), (2, 64, 256, 70, 33)], wl.BF16: [(1, 64, 64, 601, 4), (2, 64, 512, 70, 33)]}


@pytest.mark.parametrize("probe", [wl.RADEMACHER, wl.GAUSSIAN], ids=["sign", "normal"])
@pytest.mark.parametrize("wdtype,k", [(wl.FP32, 0), (wl.FP32, 1), (wl.BF16, 0), (wl.BF16, 1)],
                         ids=["fp32-narrow", "fp32-wide", "bf16-narrow", "bf16-wide"])
def test_one_position_matches_oracle(zo, oracle, wdtype, k, probe):
    L, E, H, N, B = SHAPES[wdtype][k]
    cfg = dict(n_layers=L, vocab=60, embed=E, hidden=H, wdtype=wdtype, probe=probe)
    print(f"one position {cfg} N={N} B={B}", flush=True)
    tok = wl.uniform_tokens(np.random.default_rng(H), B, 1, cfg["vocab"])
    theta = zo.new_theta(cfg)
    zo.init(cfg, theta, 3)
    td = torch.from_numpy(tok).cuda()
    ref, eps = oracle.init(cfg, 3), 1e-2
    for cache in (True, False):
        ws = zo.new_workspace(cfg, N, B, 1, probe_cache=cache)
        ws.fill_(255)
        Lp, Lm = zo.perturbed_losses(cfg, theta, 17, eps, N, td, i0=4, workspace=ws)
        ws.fill_(255)
        Lf, L0 = zo.fd_losses(cfg, theta, 17, eps, N, td, i0=4, workspace=ws)
        rp, rm = oracle.perturbed_losses(cfg, ref, 17, eps, N, tok, i0=4, as_double=True)
        rl, r0 = oracle.fd_losses(cfg, ref, 17, eps, N, tok, i0=4)
        for got, want in ((Lp, rp), (Lm, rm), (Lf, rl), (L0, np.atleast_1d(r0))):
            got = got.cpu().numpy().astype(np.float64)
            assert np.all(np.abs(got - want) <= RTOL[wdtype] * np.abs(want)), np.abs(got - want).max()
        # a state read too early or too late would not agree between the two, bit for bit
        assert torch.equal(Lp, Lf)
