"""Every tile shape of the fp32 gate and head kernels: one to four row tiles per
sign and one or two column tiles per wave, whole and partial row blocks, central
and forward differences, with the caches and packed weights and without. Every
shape sums in the same order, so a probe's losses are those of a call with that
probe alone (one row tile, one column tile), bit for bit; that one is checked
against the oracle. test_cases_reach_every_shape (no GPU) runs the launchers'
rule over the cases."""
import os
import re
import subprocess

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle  # noqa: E402
from paper_2505_17852_amd import workloads as wl  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
RTOL = 1e-5  # the fp32 path's bar against the 64-bit oracle
V = 300  # two whole vocabulary tiles and a ragged one

# (L, H, N, B): from one row tile per pass up to nine
CASES = [(1, 32, 5, 40), (1, 32, 5, 72), (1, 32, 5, 96), (1, 32, 5, 112), (1, 96, 5, 130), (1, 32, 20, 64),
         (1, 32, 20, 112), (1, 96, 20, 72), (1, 96, 20, 112), (1, 32, 70, 20), (2, 32, 70, 16), (2, 32, 70, 20),
         (2, 32, 70, 40), (1, 32, 70, 64), (2, 32, 70, 64), (2, 32, 70, 72), (2, 32, 70, 96), (1, 32, 70, 112),
         (2, 32, 70, 112), (1, 32, 100, 72), (1, 32, 100, 112), (2, 32, 100, 128)]
LENGTHS = (6, 130)  # below and above the length from which the weights are packed


def test_cases_reach_every_shape(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    exe = str(tmp_path / "f32_shapes")
    subprocess.run([HIPCC, "-O1", "-std=c++17", os.path.join(ROOT, "tests", "helpers", "f32_shapes.cpp"), "-o", exe],
                   check=True, capture_output=True)
    calls = [(L, V, H, N, B, fd, C) for L, H, N, B in CASES for fd in (0, 1) for C in LENGTHS]
    text = "\n".join(" ".join(str(x) for x in c) for c in calls)
    out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout.splitlines()
    seen = set()
    for (L, _, _, _, _, fd, _), line in zip(calls, out):
        rt, ct, rt1, ct1, head, q = (int(x) for x in line.split())
        for kind, r, c in (("gate", rt, ct), ("gate", rt1, ct1), ("head", head, 2)):
            seen.add((kind, fd, r, c, q % (2 * r if fd else r) != 0))  # the last row block of a pass is partial
    want = {("gate", fd, r, c, part) for fd in (0, 1) for r in (1, 2, 3, 4) for c in (1, 2) for part in (False, True)}
    want |= {("head", fd, r, 2, part) for fd in (0, 1) for r in (1, 2, 3, 4) for part in (False, True)}
    want -= {(k, 0, 1, c, True) for k in ("gate", "head") for c in (1, 2)}  # blocks of one row tile are whole
    assert not want - seen, sorted(want - seen)


@pytest.fixture(scope="module")
def zo():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_17852_amd import zo as z
    z.lib()
    return z


@pytest.mark.gpu
@pytest.mark.parametrize("probe", [wl.RADEMACHER, wl.GAUSSIAN], ids=["sign", "normal"])
@pytest.mark.parametrize("L,H,N,B", CASES)
def test_f32_shapes_agree(zo, L, H, N, B, probe):
    cfg = dict(n_layers=L, vocab=V, embed=32, hidden=H, wdtype=wl.FP32, probe=probe)
    eps, seed, i0 = 1e-2, 31, 2
    theta = zo.new_theta(cfg)
    zo.init(cfg, theta, 5)
    for C in LENGTHS:
        print(f"f32 shapes {cfg} N={N} B={B} C={C}", flush=True)
        tok = wl.uniform_tokens(np.random.default_rng(B), B, C, V)
        td = torch.from_numpy(tok).cuda()
        for f, ref in ((zo.perturbed_losses, oracle.perturbed_losses), (zo.fd_losses, oracle.fd_losses)):
            fd = f is zo.fd_losses
            a, b = f(cfg, theta, seed, eps, N, td, i0=i0)
            with pytest.raises(zo.ZoError) as e:
                f(cfg, theta, seed, eps, N, td, i0=i0, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
            fewest = int(re.search(r"< (\d+) required", str(e.value)).group(1))
            ws = torch.full((fewest,), 255, dtype=torch.uint8, device="cuda")
            a2, b2 = f(cfg, theta, seed, eps, N, td, i0=i0, workspace=ws)
            assert torch.equal(a2, a) and torch.equal(b2, b)
            for n in (0, N // 2, N - 1):
                s, t = f(cfg, theta, seed, eps, 1, td, i0=i0 + n)
                assert torch.equal(s, a[n:n + 1]) and torch.equal(t, b if fd else b[n:n + 1])
            if C == LENGTHS[0] and not fd:  # the two-stream form: the same products, other roundings
                p = f(cfg, theta, seed, eps, N, td, i0=i0, products=zo.PRODUCTS_SPLIT)
                q = f(cfg, theta, seed, eps, 1, td, i0=i0 + N - 1, products=zo.PRODUCTS_SPLIT)
                for x, y, z in zip(p, q, (a, b)):
                    assert torch.equal(y, x[N - 1:]) and torch.all((x - z).abs() <= RTOL * z.abs())
            if C == LENGTHS[0]:
                kw = {} if fd else dict(as_double=True)
                want = ref(cfg, oracle.init(cfg, 5), seed, eps, 1, tok, i0=i0 + N - 1, **kw)
                for got, w in ((a[N - 1], want[0]), (b[0] if fd else b[N - 1], want[1])):
                    assert abs(float(got) - np.ravel(w)[0]) <= RTOL * np.ravel(w)[0]
