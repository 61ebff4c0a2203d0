"""fp32 losses do not depend on the workspace, bit for bit: a full one (caches and
the longest chunk), the smallest reported one, one of a larger call, and the
fewest bytes that the call takes (no caches, chunks of two timesteps)."""
import re

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


@pytest.mark.parametrize("probe", [wl.RADEMACHER, wl.GAUSSIAN], ids=["sign", "normal"])
# (L, V, E, H, N, B, C): chunks of 8 and more, packed weights; C below a chunk, read in place
@pytest.mark.parametrize("shape", [(2, 300, 96, 160, 5, 20, 67), (3, 1000, 64, 128, 40, 64, 43), (1, 77, 32, 64, 3, 17, 5)],
                         ids=["ragged", "rows", "short"])
def test_f32_losses_do_not_depend_on_the_workspace(zo, shape, probe):
    L, V, E, H, N, B, C = shape
    cfg = dict(n_layers=L, vocab=V, embed=E, hidden=H, wdtype=wl.FP32, probe=probe)
    theta = zo.new_theta(cfg)
    zo.init(cfg, theta, 6)
    rng = np.random.default_rng(C)
    td = torch.from_numpy(wl.uniform_tokens(rng, B, C, V)).cuda()
    md = torch.from_numpy((rng.random((B, C)) < 0.7).astype(np.uint8)).cuda()
    for f in (zo.perturbed_losses, zo.fd_losses):
        with pytest.raises(zo.ZoError) as e:
            f(cfg, theta, 9, 1e-2, N, td, md, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
        fewest = int(re.search(r"< (\d+) required", str(e.value)).group(1))
        sizes = [zo.workspace_bytes(cfg, N, B, C), zo.workspace_bytes_min(cfg, N, B, C),
                 zo.workspace_bytes(cfg, N + 3, B + 20, C + 9), fewest]
        print(f"f32 workspaces {cfg} N={N} B={B} C={C} {f.__name__} bytes {sizes}", flush=True)
        assert fewest <= min(sizes[:3])
        want = None
        for size in sizes:
            ws = torch.full((size,), 255, dtype=torch.uint8, device="cuda")
            got = f(cfg, theta, 9, 1e-2, N, td, md, workspace=ws)
            want = want or got
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), size
            assert torch.all(torch.isfinite(got[0]))
