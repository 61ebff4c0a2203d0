"""Initialisation and the normal-probe update of more parameters than the threads
of one grid dimension cover (four a thread, 2^34): their last parameters and
those around the 2^34th against the probe stream."""
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


def test_init_and_normal_update_past_2_34_parameters(zo):
    cfg = dict(n_layers=1, vocab=1048583, embed=8192, hidden=8192, wdtype=wl.BF16, probe=wl.GAUSSIAN)
    P, eps, lr, seed, i0 = zo.param_count(cfg), 1e-3, 1e-1, 5, 7
    assert P > 1 << 34
    print(f"wide update P={P}", flush=True)
    theta = torch.full((P,), float("nan"), dtype=torch.bfloat16, device="cuda")
    zo.init(cfg, theta, 1)
    n = 4096
    at = [0, (1 << 34) - n // 2, P - n]
    old = [theta[j:j + n].float() for j in at]
    for x in old:
        assert torch.all(x.abs() <= 8192 ** -0.5) and x.std() > 0.5 * 8192 ** -0.5
    lp, lm = (torch.tensor(v, device="cuda") for v in ([2.003, 2.001], [2.001, 2.002]))
    zo.update(cfg, theta, seed, eps, lr, lp, lm, i0=i0)
    for j, x in zip(at, old):
        want = x.double()
        for k in range(2):
            c = lr / 2 * (lp[k].double() - lm[k].double()) / (2 * eps)
            want -= c * zo.debug_probe(wl.GAUSSIAN, seed, i0 + k, j, n).double()
        # two fp32 sums, then the bf16 rounding of the result
        assert torch.all((theta[j:j + n].double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-6)
