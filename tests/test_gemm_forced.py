"""The GEMM's kernels above 128 tokens at the edges that the automatic choice leaves to the few-token kernel with several token tiles: forced (family 2),
so that spread starts, stages of 128 k, touched weights and residuals of odd rows run where they are listed.  On the CPU: what the entry points
launch for these calls, asked through them."""
import os
import shutil
import subprocess
from collections import namedtuple

import numpy as np
import pytest

from paper_2605_25655_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
PLAIN, GATE_UP = 0, 2
FORCED = 2
Product = namedtuple("Product", "config cut touching rows tiles_m")

# Two token tiles that start spread over k: whole tiles and ranges, one row of tiles, fewer k-tiles than rows of tiles
SPREAD_STARTS = [(129, 4096, 4096), (256, 392, 1216), (130, 16, 640), (255, 2000, 448)]
# Stages of 128 k: a K that ends in a stage's first and last piece and inside, one to ten stages, whole tiles and ranges
LONG_STAGES = [(129, 1000, 1032), (256, 1111, 1144), (300, 2003, 8 * 129 + 128), (270, 1030, 8 * 95), (250, 257, 2000)]
# Two workgroups per compute unit: one and two k-tiles, a single token row of the last tile
SHORT_K = [(255, 2000, 64), (200, 300, 136), (140, 100, 256)]
# Idle compute units that touch the weights ahead: as few tiles as it takes, tiles that do not divide by the XCDs
TOUCHED = [(129, 453, 512), (385, 200, 1472), (385, 1300, 448), (385, 1500, 1280)]
# Residuals of rows whose last outputs do not fill a quad, and fewer than four of them
ODD_ROWS = [(333, 1001, 1384), (300, 3, 328), (150, 1, 264), (160, 272, 520)]
EVERY = SPREAD_STARTS + LONG_STAGES + SHORT_K + TOUCHED + ODD_ROWS


def products(tmp_path, calls):
    """What launch_gemm runs for each (family, epilogue, M, N, K)."""
    exe = str(tmp_path / "product_driver")
    csrc = os.path.join(ROOT, "paper_2605_25655_amd", "csrc")
    res = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Wno-unused-command-line-argument",
                          "-Wl,--wrap=_ZN3thi11launch_gemmERKNS_8GemmArgsEiiP12ihipStream_t", "-o", exe, os.path.join(csrc, "api.hip"),
                          os.path.join(csrc, "plan.hip"), "-x", "hip", os.path.join(ROOT, "tests", "sanitize", "api_stubs.cpp"),
                          os.path.join(ROOT, "tests", "plan", "product_driver.cpp")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    text = "".join("%d %d %d %d %d\n" % c for c in calls)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    got = [Product(f[0], *map(int, f[1:])) for f in (line.split() for line in out if line)]
    assert len(got) == len(calls)
    return got


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")
def test_these_calls_run_the_kernels_they_are_listed_for(tmp_path):
    picks = dict(zip(EVERY, products(tmp_path, [(FORCED, PLAIN, *s) for s in EVERY])))
    assert all(p.config in ("FEW128", "DEEP", "SMALL") for p in picks.values()), picks
    spread = [picks[s] for s in SPREAD_STARTS]      # (FEW128 with two token tiles and whole stages of 64 k)
    assert all(p.config == "FEW128" and s[0] <= 256 and s[2] % 64 == 0 for s, p in zip(SPREAD_STARTS, spread)), spread
    assert any(p.cut for p in spread) and any(not p.cut for p in spread)
    assert all(picks[s].config == "DEEP" for s in LONG_STAGES) and all(picks[s].config == "SMALL" for s in SHORT_K), picks
    assert any(picks[s].cut for s in LONG_STAGES) and any(not picks[s].cut for s in LONG_STAGES)
    assert all(picks[s].touching > 0 and picks[s].touching % 8 == 0 and not picks[s].cut for s in TOUCHED), picks
    # ... and the automatic choice, which runs them as the few-token kernel's token tiles
    assert all(p.config == "MID" and p.tiles_m > 1 for p in products(tmp_path, [(0, PLAIN, *s) for s in EVERY]))


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", EVERY)
def test_forced_gemm_kernels(M, N, K):
    import torch

    import oracle
    import paper_2605_25655_amd as thi
    from tests.gpu_common import Runner, to_dev, to_host
    from tests.parity import check
    print(f"[case] GEMM forced M={M} N={N} K={K}", flush=True)
    x, w, g = synth.random_problem(16000 + M + N + K, M, N, K)
    rng = np.random.Generator(np.random.Philox(key=16100 + M + N + K))
    res = rng.standard_normal((M, N)).astype(np.float16)
    hd = 8
    n_rot = N // 2 // hd * hd
    pos = rng.integers(0, 4096, size=M).astype(np.int32)
    th = (10000.0 ** (-np.arange(0, hd, 2, dtype=np.float64) / hd)).astype(np.float32)
    rows = np.unique(np.concatenate([synth.sample_rows(61, M, 8), [0, 127, 128, M - 1]]))
    r = Runner(M, K, K, N)
    xd, wd, gd, rd = to_dev(x), to_dev(w), to_dev(g), to_dev(res)
    prev = thi.thi_set_kernel_family(FORCED)
    try:
        a = [to_host(r.linear(xd, wd)) for _ in range(3)]
        b = [to_host(r.linear_residual(xd, wd, rd)) for _ in range(2)] + [to_host(r.linear_residual(xd, wd, rd, in_place=True))]
        c = to_host(r.rmsnorm_qkv_rope(xd, gd, 1e-6, wd, torch.from_numpy(pos).cuda(), torch.from_numpy(th).cuda(), n_rot, hd))
    finally:
        thi.thi_set_kernel_family(prev)
    for runs in (a, b):
        assert all(np.array_equal(runs[0].view(np.uint16), v.view(np.uint16)) for v in runs[1:]), "not reproducible, or another result in place"
    for out in (a[0], b[0], c):
        assert np.isfinite(out.astype(np.float32)).all()
    y, s = oracle.linear(x[rows], w)
    check(a[0][rows], y, s, "linear", argmax=False)
    y, s = oracle.linear_residual(x[rows], w, res[rows])
    check(b[0][rows], y, s, "linear + residual", argmax=False)
    y, s = oracle.rmsnorm_qkv_rope(x[rows], g, 1e-6, w, pos[rows], th, n_rot, hd)
    check(c[rows], y, s, "rmsnorm_qkv_rope", argmax=False)
