"""Calls whose head takes more workgroups than one grid dimension holds (their
threads past 2^32): the losses of a probe are those of a call with that probe
alone, bit for bit."""
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


# (wdtype, E = H, N, B): 2 N B rows and 2 timesteps by 131,072 words: fp32 16,400 blocks of 32 rows
# x 1,024 tiles of 256 threads, bf16 16,400 of 64 rows x 512 tiles of 512
@pytest.mark.parametrize("wdtype,H,N,B", [(wl.FP32, 32, 8200, 16), (wl.BF16, 64, 8200, 32)], ids=["fp32", "bf16"])
def test_head_of_more_workgroups_than_one_dimension(zo, wdtype, H, N, B):
    cfg = dict(n_layers=1, vocab=131072, embed=H, hidden=H, wdtype=wdtype, probe=wl.RADEMACHER)
    print(f"wide grid {cfg} N={N} B={B}", flush=True)
    theta = zo.new_theta(cfg)
    zo.init(cfg, theta, 1)
    td = torch.from_numpy(wl.uniform_tokens(np.random.default_rng(0), B, 2, cfg["vocab"])).cuda()
    Lp, Lm = zo.perturbed_losses(cfg, theta, 5, 1e-2, N, td, i0=3)
    for n in (0, N // 2, N - 1):
        a, b = zo.perturbed_losses(cfg, theta, 5, 1e-2, 1, td, i0=3 + n)
        assert torch.equal(a, Lp[n:n + 1]) and torch.equal(b, Lm[n:n + 1])
    assert torch.all(torch.isfinite(Lp)) and torch.all(torch.isfinite(Lm))
