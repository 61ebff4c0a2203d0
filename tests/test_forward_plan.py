"""The host side of the forward calls (workspace plans, buffers and launch
order), without a GPU: zo_api.hip and k_forward.hip built for the host with
their kernel launchers replaced by checks (tests/helpers/forward_plan_driver.cpp).
Every buffer of every launch lies inside the workspace and apart from the
others, and no launch writes a state that its other workgroups still read."""
import os
import subprocess

import pytest

from paper_2505_17852_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_17852_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, " ".join(cmd) + "\n" + r.stdout[-2000:] + r.stderr[-4000:]


@pytest.fixture(scope="module")
def calls(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("plan")
    objs = []
    for src in ("zo_api.hip", "zo_profile.hip", "k_forward.hip"):
        objs.append(str(d / (src + ".o")))
        run([HIPCC, "-std=c++17", "-O1", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
             "-packed-fp32-ops", "-c", os.path.join(CSRC, src), "-o", objs[-1]])
    objs.append(str(d / "driver.o"))
    run([HIPCC, "-std=c++17", "-O1", "-x", "c++", "-I/opt/rocm/include", "-D__HIP_PLATFORM_AMD__", "-c",
         os.path.join(ROOT, "tests", "helpers", "forward_plan_driver.cpp"), "-o", objs[-1]])
    exe = str(d / "forward_plan")
    run([HIPCC, *objs, "-L/opt/rocm/lib", "-lrocprofiler-sdk-roctx", "-Wl,-rpath,/opt/rocm/lib", "-o", exe])

    def call(lines):
        """lines: (cfg, fd, N, B, C, ws_bytes); per line (status, bytes used, steps per chunk, caches)."""
        text = "".join(" ".join(str(x) for x in (c["n_layers"], c["vocab"], c["embed"], c["hidden"], c["wdtype"],
                                                 c["probe"], fd, N, B, C, ws)) + "\n" for c, fd, N, B, C, ws in lines)
        r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-2000:]
        out = [tuple(int(x) for x in line.split()) for line in r.stdout.splitlines()]
        assert len(out) == len(lines)
        for line, o in zip(lines, out):
            assert o[4] == 0, f"{line}: {o[4]} violations\n{r.stderr[-2000:]}"
        return [o[:4] for o in out]

    return call


@pytest.fixture(scope="module")
def zo():
    from paper_2505_17852_amd import zo as z
    if not os.path.exists(z.LIB_PATH):
        from paper_2505_17852_amd import build
        build.build()
    z.lib()
    return z


def model(L, V, E, H, wdtype, probe):
    return dict(n_layers=L, vocab=V, embed=E, hidden=H, wdtype=wdtype, probe=probe)


@pytest.mark.parametrize("wdtype", [wl.FP32, wl.BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("C", [1, 2, 3, 17, 70])
def test_states_are_not_written_while_read(calls, zo, C, wdtype):
    """Among them C = 1, where the chunk has one slot for the top layer."""
    lines = []
    for L in (1, 2, 9):
        for probe in (wl.RADEMACHER, wl.GAUSSIAN):
            cfg = model(L, 300, 64, 192, wdtype, probe)
            for N, B in ((1, 1), (3, 33)):
                for ws in (zo.workspace_bytes(cfg, N, B, C), zo.workspace_bytes_min(cfg, N, B, C)):
                    lines += [(cfg, fd, N, B, C, ws) for fd in (0, 1)]
                lines.append((cfg, 2, N, B, C, 0))
    assert all(o[0] == zo.ZO_OK for o in calls(lines))
