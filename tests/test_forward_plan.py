"""The host side of the forward calls (workspace plans, buffers and launch
order), without a GPU: zo_api.hip and k_forward.hip built for the host with
their kernel launchers replaced by checks (tests/helpers/forward_plan_driver.cpp).
Every buffer of every launch lies inside the workspace and apart from the
others, and no launch writes a state that its other workgroups still read."""
import ctypes
import math
import os
import random
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


def _draw(rng, wdtype):
    g = 64 if wdtype == wl.BF16 else 32

    def lg(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    cfg = model(rng.choice([1, 2, 3, 6]), lg(1, 50000), g * lg(1, 20), g * lg(1, 20), wdtype,
                rng.choice([wl.RADEMACHER, wl.GAUSSIAN]))
    return cfg, (lg(1, 600), lg(1, 300), lg(1, 60))


# (cfg, larger call, smaller call): N, B, C
REUSE = {
    wl.BF16: [(model(2, 7401, 832, 1088, wl.BF16, wl.RADEMACHER), (38, 166, 27), (37, 159, 27)),
              (model(4, 1536, 1024, 64, wl.BF16, wl.GAUSSIAN), (28, 6, 61), (17, 6, 41)),
              (model(2, 10000, 512, 768, wl.BF16, wl.RADEMACHER), (33, 160, 32), (32, 160, 32)),
              (model(2, 10000, 512, 768, wl.BF16, wl.GAUSSIAN), (33, 160, 32), (32, 160, 32))],
    wl.FP32: [(model(2, 256, 128, 256, wl.FP32, wl.RADEMACHER), (1, 81, 256), (1, 80, 256)),
              (model(1, 128, 32, 32, wl.FP32, wl.GAUSSIAN), (1, 32, 64), (1, 32, 9))],
}


@pytest.mark.parametrize("wdtype", list(REUSE), ids=lambda w: "bf16" if w == wl.BF16 else "fp32")
def test_a_workspace_holds_every_smaller_call(calls, zo, wdtype):
    """A workspace sized for a call also holds every call with at most as many
    probes, sequences and positions, with the caches that the smaller call has
    in a workspace of its own."""
    rng = random.Random(5)
    pairs = list(REUSE[wdtype])
    for _ in range(1000):
        cfg, big = _draw(rng, wdtype)
        small = list(big)
        for k in range(3):
            if rng.random() < 0.6:  # a little less, or anything less
                small[k] = max(1, big[k] - rng.randint(0, 3)) if rng.random() < 0.5 else rng.randint(1, big[k])
        pairs.append((cfg, big, tuple(small)))
    lines, own = [], []
    for cfg, big, small in pairs:
        for size in (zo.workspace_bytes, zo.workspace_bytes_min):
            assert size(cfg, *small) <= size(cfg, *big), (cfg, big, small)
            for fd in (0, 1):
                lines.append((cfg, fd, *small, size(cfg, *big)))
                own.append((cfg, fd, *small, size(cfg, *small)))
    for line, mine, a, b in zip(lines, own, calls(lines), calls(own)):
        assert a[0] == b[0] == zo.ZO_OK, (line, a, b)
        assert a[3] & b[3] & 3 == b[3] & 3, (line, mine, a, b)


def _plain(cfg, N, B, C):
    """Bytes of a call with fp32 activations (fp16 with bf16 weights), batches
    padded to 32 or 128 (twice that for forward differences) and chunks of 16
    timesteps: the smallest workspace before the fp32 states were stored in three
    parts and the bf16 tiles got smaller, and the no-alloc entry point's account."""
    L, V, E, H = cfg["n_layers"], cfg["vocab"], cfg["embed"], cfg["hidden"]
    b16 = cfg["wdtype"] == wl.BF16
    g, vt, el = (128, 256, 2) if b16 else (32, 128, 4)
    T, nvt, size = min(C, 16), (V + vt - 1) // vt, 0
    pg = sum(4 * H * ((E if l == 0 else H) + H) for l in range(L)) + nvt * vt * H
    for M in (2 * N * ((B + g - 1) // g * g), (N + 1) * ((B + 2 * g - 1) // (2 * g) * (2 * g))):
        parts = [(1 if b16 else T) * M * E * el, (L - 1) * 2 * M * H * el, T * M * H * el, L * M * H * 4,
                 L * N * 4 * H * 4, N * V * 4, nvt * T * M * 4, nvt * T * M * 4, T * M * 4, M * 8, pg * 2 if b16 else 0]
        size = max(size, sum((p + 255) // 256 * 256 for p in parts))
    return size


def test_smallest_f32_workspace_needs_no_caches(calls, zo):
    """The smallest fp32 workspace leaves out the packed weights and the sign
    words (the forward runs without): calls of at least a chunk of positions run
    in as many bytes as before either was stored, and the size reported is at
    most 32 MiB above that."""
    assert _plain(wl.model_cfg("c2"), 32, 64, 256) == 119078912  # 113.6 MiB
    cases = [(model(2, 50000, 512, 1024, wl.FP32, wl.RADEMACHER), 96, 32, 16),
             (model(6, 50000, 1024, 2048, wl.FP32, wl.RADEMACHER), 64, 16, 64)]
    rng = random.Random(8)
    while len(cases) < 400:
        cfg, (N, B, C) = _draw(rng, wl.FP32)
        cases.append((cfg, N, B, C + 15))
    for cfg, N, B, C in cases:
        size, plain = zo.workspace_bytes_min(cfg, N, B, C), _plain(cfg, N, B, C)
        assert plain <= size <= plain + (32 << 20), (cfg, N, B, C, size, plain)
    lines = [(cfg, fd, N, B, C, _plain(cfg, N, B, C)) for cfg, N, B, C in cases for fd in (0, 1)]
    out = calls(lines)
    assert all(o[0] == zo.ZO_OK for o in out)
    # and a full one holds both caches
    full = calls([(cfg, fd, N, B, C, zo.workspace_bytes(cfg, N, B, C)) for cfg, N, B, C in cases for fd in (0, 1)])
    for line, o in zip(lines, full):
        cfg, C = line[0], line[4]
        packs = C * (cfg["embed"] + cfg["hidden"]) // 32 >= 256
        assert o[0] == zo.ZO_OK and o[3] == (1 if cfg["probe"] == wl.RADEMACHER else 2) + 4 * packs, (line, o)


@pytest.mark.parametrize("wdtype", [wl.FP32, wl.BF16], ids=["fp32", "bf16"])
def test_noalloc_array_holds_every_call_its_account_admits(calls, zo, wdtype):
    """zo_perturbed_losses_noalloc takes a call exactly when its account is at most
    ZO_NOALLOC_WORKSPACE_BYTES, and then finds room in the array: at the largest
    number of probes the account admits, and refused at one more."""
    rng = random.Random(11)
    shapes = [(model(1, 3, 32, 4096, wl.FP32, wl.RADEMACHER), 32, 1), (model(64, 3, 32, 512, wl.FP32, wl.GAUSSIAN), 32, 9),
              (model(1, 100, 32, 32, wl.FP32, wl.RADEMACHER), 32, 64)] if wdtype == wl.FP32 else []
    while len(shapes) < 400:
        cfg, (_, B, C) = _draw(rng, wdtype)
        cfg["n_layers"] = rng.choice([1, 2, 3, 6, 20, 64])
        shapes.append((cfg, B, rng.choice([1, 2, 3, C])))
    lines, want = [], []
    for cfg, B, C in shapes:
        lo, hi = 0, 1 << 20  # account(lo) fits, account(hi) does not
        while hi - lo > 1:
            n = (lo + hi) // 2
            lo, hi = (n, hi) if _plain(cfg, n, B, C) <= zo.NOALLOC_WORKSPACE_BYTES else (lo, n)
        for n in (lo, hi) if lo else (hi,):
            lines.append((cfg, 2, n, B, C, 0))
            want.append(zo.ZO_OK if n == lo else zo.ZO_ENOMEM)
    assert want.count(zo.ZO_OK) > 250
    for line, st, o in zip(lines, want, calls(lines)):
        assert o[0] == st, (line, o)


def test_bf16_matrices_beyond_32_bit_offsets_are_refused(calls, zo):
    """A packed matrix of 4 GiB and more (the head with its vocabulary in whole
    256-word tiles, or a gate matrix) is ZO_ESHAPE; the largest below it runs.
    fp32 weights have no such bound."""
    big = [(1, 262144, 64, 8192), (1, 261889, 64, 8192), (1, 100, 64, 23232), (1, 100, 65536, 8192)]
    below = [(1, 261888, 64, 8192), (1, 100, 64, 23104), (1, 100, 65472, 8192)]
    for shapes, wdtype, want in ((big, wl.BF16, zo.ZO_ESHAPE), (below, wl.BF16, zo.ZO_OK), (big, wl.FP32, zo.ZO_OK)):
        cfgs = [model(*s, wdtype, p) for s in shapes for p in (wl.RADEMACHER, wl.GAUSSIAN)]
        lines = [(c, fd, 1, 3, 2, zo.workspace_bytes(c, 1, 3, 2)) for c in cfgs for fd in (0, 1)]
        assert all(o[0] == want for o in calls(lines)), (shapes, wdtype)


def test_sign_words_past_32_bit_offsets_are_not_cached(calls, zo):
    """From 2^35 parameters on a probe's words take 4 GiB: the bf16 forward
    regenerates them, whatever the workspace; below, a full one holds them."""
    for L, cached in ((18, 1), (19, 0)):  # 33.1 and 35.0 G parameters; 2^35 is 34.4 G
        cfg = model(L, 2000, 64, 15360, wl.BF16, wl.RADEMACHER)
        assert (zo.param_count(cfg) < 1 << 35) == bool(cached)
        full, small = zo.workspace_bytes(cfg, 1, 3, 2), zo.workspace_bytes_min(cfg, 1, 3, 2)
        assert (full > small) == bool(cached)
        offset = zo.lib().zo_probe_bits_offset(ctypes.byref(zo._cfg(cfg)), 1, 3, 2)
        assert (offset > 0) == bool(cached)
        for ws in (full, full + (8 << 30)):
            (o,) = calls([(cfg, 0, 1, 3, 2, ws)])
            assert o[0] == zo.ZO_OK and o[3] == cached, (L, ws, o)
