"""The bf16 path's tile shapes (256, 128 and 64 rows, and a launch that ends in
64-row tiles): every shape sums in the same order, so the losses of a probe do
not depend on the number of probes beside it (which picks the shape), bit for
bit; one probe's losses are checked against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import oracle  # noqa: E402
from paper_2505_17852_amd import workloads as wl  # noqa: E402

RTOL = 2e-5  # losses of small models against the 64-bit oracle: fp16 operands, errors averaged over B C positions


@pytest.fixture(scope="module")
def zo():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_17852_amd import zo as z
    z.lib()
    return z


# (N, B, fd): with 256 hidden units, central: 256 rows per tile (64 x 128), 128
# (64 x 64), 64 (9 x 33); forward: 128 rows with a rest in 64-row tiles (64 x
# 128), 64 (3 x 1). A call with one probe takes 64-row tiles.
CASES = [(64, 128, False), (64, 64, False), (9, 33, False), (64, 128, True), (3, 1, True)]


@pytest.mark.parametrize("probe,eps,cache", [(wl.RADEMACHER, 1e-2, True), (wl.RADEMACHER, 1e-4, False),
                                             (wl.GAUSSIAN, 1e-2, True), (wl.GAUSSIAN, 1e-4, True),
                                             (wl.GAUSSIAN, 1e-2, False)],
                         ids=["sign", "sign-2stream-regen", "normal", "normal-2stream", "normal-regen"])
@pytest.mark.parametrize("N,B,fd", CASES)
def test_tiles_agree(zo, N, B, fd, probe, eps, cache):
    cfg = dict(n_layers=2, vocab=300, embed=64, hidden=256, wdtype=wl.BF16, probe=probe)
    C, i0 = 2, 5
    print(f"bf16 tiles N={N} B={B} fd={fd} probe={probe} eps={eps} cache={cache}", flush=True)
    tok = wl.uniform_tokens(np.random.default_rng(B), B, C, cfg["vocab"])
    td = torch.from_numpy(tok).cuda()
    theta = zo.new_theta(cfg)
    zo.init(cfg, theta, 5)

    def losses(n, first):
        ws = zo.new_workspace(cfg, n, B, C, probe_cache=cache)
        f = zo.fd_losses if fd else zo.perturbed_losses
        return f(cfg, theta, 31, eps, n, td, i0=i0 + first, workspace=ws)

    a, b = losses(N, 0)
    for n in (0, N // 2, N - 1):
        s, t = losses(1, n)
        assert torch.equal(s, a[n:n + 1])
        assert torch.equal(t, b if fd else b[n:n + 1])
    ref = oracle.init(cfg, 5)
    if fd:
        rs, rt = oracle.fd_losses(cfg, ref, 31, eps, 1, tok, i0=i0)
    else:
        rs, rt = oracle.perturbed_losses(cfg, ref, 31, eps, 1, tok, i0=i0, as_double=True)
    assert abs(float(a[0]) - np.ravel(rs)[0]) <= RTOL * np.ravel(rs)[0]
    assert abs(float(b[0]) - np.ravel(rt)[0]) <= RTOL * np.ravel(rt)[0]
