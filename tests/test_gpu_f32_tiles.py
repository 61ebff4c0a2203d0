"""fp32 products as sums of bf16 matrix products against the oracle: batches around
multiples of 16 rows, K tiles that do not fill a stage, small and ragged
vocabularies, for sign and normal probes, central and forward differences. Calls
as small as these take one row tile per workgroup; the other tile shapes are in
test_gpu_f32_shapes.py."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import oracle  # noqa: E402
from paper_2505_17852_amd import workloads as wl  # noqa: E402

# The oracle runs in 64 bits; a loss is off by its fp32 rounding and the fp32
# sums behind it (the bar of the fp32 path's other tests).
RTOL = 1e-5


@pytest.fixture(scope="module")
def zo():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_17852_amd import zo as z
    z.lib()
    return z


def say(*a):
    print(*a, flush=True)


# (B, E, H, V, C): 1, 1, 2, 3, 4, 5 and 9 row tiles per pass; K tiles
# of 1 + 1 up to 5 + 3; vocabularies of 1, 128, 129 and 300
SHAPES = [(1, 32, 32, 1, 3), (16, 32, 64, 128, 2), (17, 64, 32, 129, 2), (47, 96, 96, 40, 3), (64, 160, 96, 300, 2),
          (65, 32, 96, 77, 2), (130, 64, 64, 50, 2)]


@pytest.mark.parametrize("probe", [wl.RADEMACHER, wl.GAUSSIAN], ids=["sign", "normal"])
@pytest.mark.parametrize("shape", SHAPES, ids=[f"B{s[0]}" for s in SHAPES])
def test_tile_shapes_match_oracle(zo, shape, probe):
    B, E, H, V, C = shape
    cfg = dict(n_layers=2, vocab=V, embed=E, hidden=H, wdtype=wl.FP32, probe=probe)
    N, eps, i0 = 3, 1e-2, 2
    say(f"f32 tiles {cfg} N={N} B={B} C={C}")
    rng = np.random.default_rng(B)
    tok = wl.uniform_tokens(rng, B, C, V)
    theta = zo.new_theta(cfg)
    zo.init(cfg, theta, 5)
    ref = oracle.init(cfg, 5)
    td = torch.from_numpy(tok).cuda()
    Lp, Lm = zo.perturbed_losses(cfg, theta, 31, eps, N, td, i0=i0)
    L, L0 = zo.fd_losses(cfg, theta, 31, eps, N, td, i0=i0)
    rp, rm = oracle.perturbed_losses(cfg, ref, 31, eps, N, tok, i0=i0, as_double=True)
    rl, r0 = oracle.fd_losses(cfg, ref, 31, eps, N, tok, i0=i0)
    for got, want in ((Lp, rp), (Lm, rm), (L, rl), (L0, np.atleast_1d(r0))):
        got = got.cpu().numpy()
        assert np.all(np.abs(got - want) <= RTOL * np.abs(want) + 1e-7), (got, want)
    # every shape sums in the same order: the + passes of the two estimators agree bit for bit,
    # and so does a slice of the probes
    assert torch.equal(Lp, L)
    sp, _ = zo.perturbed_losses(cfg, theta, 31, eps, 1, td, i0=i0 + 1)
    assert torch.equal(sp, Lp[1:2])


def test_regenerated_sign_words_match_the_workspace(zo):
    """A vocabulary and embedding too large for the fixed scratch to hold the
    probes' sign words: the kernels regenerate them, bit for bit."""
    cfg = dict(n_layers=1, vocab=40000, embed=512, hidden=32, wdtype=wl.FP32, probe=wl.RADEMACHER)
    N, B, C = 84, 2, 2
    assert N * zo.param_count(cfg) // 8 > zo.NOALLOC_WORKSPACE_BYTES * 3 // 2  # the words alone exceed the scratch
    say(f"f32 regenerated signs {cfg} N={N} B={B} C={C}")
    theta = zo.new_theta(cfg)
    zo.init(cfg, theta, 8)
    td = torch.from_numpy(wl.uniform_tokens(np.random.default_rng(1), B, C, cfg["vocab"])).cuda()
    Lp, Lm = torch.empty(N, device="cuda"), torch.empty(N, device="cuda")
    zo.perturbed_losses_noalloc(cfg, theta, 4, 1e-2, N, td, None, Lp, Lm)
    rp, rm = zo.perturbed_losses(cfg, theta, 4, 1e-2, N, td)
    assert torch.equal(Lp, rp) and torch.equal(Lm, rm) and torch.all(torch.isfinite(Lp))
