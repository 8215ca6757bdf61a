"""Rotary embedding of heads wider than the 256 columns that the table in the workspace holds: between 33 and 64 tokens the stream-K decode kernel
rotates them itself, so such calls stay with it whatever the other kernels would take."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2605_25655_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SHAPES = [(33, 3072, 2048), (34, 12288, 4096), (48, 12288, 4096), (64, 12288, 4096), (48, 10240, 8192), (64, 15360, 5120)]


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")
def test_wide_heads_are_accepted_up_to_64_tokens(tmp_path):
    exe = str(tmp_path / "rope_heads")
    csrc = os.path.join(ROOT, "paper_2605_25655_amd", "csrc")
    res = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Wno-unused-command-line-argument", "-o", exe,
                          os.path.join(csrc, "api.hip"), os.path.join(csrc, "plan.hip"), "-x", "hip",
                          os.path.join(ROOT, "tests", "sanitize", "api_stubs.cpp"), os.path.join(ROOT, "tests", "plan", "rope_heads.cpp")],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    calls = [(M, N, K, hd) for M, N, K in SHAPES for hd in (512, 1024)] + [(32, 12288, 4096, 512), (48, 12288, 4096, 256), (65, 12288, 4096, 512), (65, 12288, 4096, 256)]
    text = "".join("%d %d %d %d %d\n" % (M, N, K, 1024, hd) for M, N, K, hd in calls)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    got = [tuple(map(int, line.split())) for line in out if line]
    assert got[:len(SHAPES) * 2] == [(0, 1)] * (len(SHAPES) * 2), list(zip(calls, got))
    # up to 32 tokens any head; at 256 columns the pass that fills the table and a GEMM kernel; above 64 tokens no kernel without the table
    assert got[len(SHAPES) * 2:] == [(0, 1), (0, 2), (2, 0), (0, 2)], list(zip(calls, got))[len(SHAPES) * 2:]


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(34, 3072, 2048), (48, 12288, 4096), (64, 6144, 8192)])
@pytest.mark.parametrize("hd", [256, 512])
def test_wide_heads_between_33_and_64_tokens(M, N, K, hd):
    import torch

    import oracle
    from tests.gpu_common import Runner, to_dev, to_host
    from tests.parity import check
    print(f"[case] wide heads M={M} N={N} K={K} head_dim={hd}", flush=True)
    x, w, g = synth.random_problem(15000 + M + N + K, M, N, K)
    n_rot = N // 2 // hd * hd
    pos = np.random.Generator(np.random.Philox(key=15100 + M + N + K)).integers(0, 4096, size=M).astype(np.int32)
    th = (10000.0 ** (-np.arange(0, hd, 2, dtype=np.float64) / hd)).astype(np.float32)
    r = Runner(M, K, K, N)
    got = to_host(r.rmsnorm_qkv_rope(to_dev(x), to_dev(g), 1e-6, to_dev(w), torch.from_numpy(pos).cuda(), torch.from_numpy(th).cuda(), n_rot, hd))
    rows = np.unique(np.concatenate([synth.sample_rows(51, M, 8), [0, M - 1]]))
    y, s = oracle.rmsnorm_qkv_rope(x[rows], g, 1e-6, w, pos[rows], th, n_rot, hd)
    check(got[rows], y, s, "rmsnorm_qkv_rope", argmax=False)
    assert np.isfinite(got.astype(np.float32)).all()


@pytest.mark.gpu
@pytest.mark.parametrize("M", [48, 64])
def test_narrow_heads_on_the_streamk_kernel(M):
    """Three and four token tiles of a shape whose automatic choice rotates through the table of the RMSNorm pass: the rotation inside the kernel."""
    import torch

    import oracle
    import paper_2605_25655_amd as thi
    from tests.gpu_common import Runner, to_dev, to_host
    from tests.parity import check
    N, K, hd = 12288, 4096, 64
    print(f"[case] narrow heads, stream-K M={M} N={N} K={K}", flush=True)
    x, w, g = synth.random_problem(15200 + M, M, N, K)
    n_rot = N // 2
    pos = np.random.Generator(np.random.Philox(key=15300 + M)).integers(0, 4096, size=M).astype(np.int32)
    th = (10000.0 ** (-np.arange(0, hd, 2, dtype=np.float64) / hd)).astype(np.float32)
    r = Runner(M, K, K, N)
    prev = thi.thi_set_kernel_family(1)
    try:
        got = to_host(r.rmsnorm_qkv_rope(to_dev(x), to_dev(g), 1e-6, to_dev(w), torch.from_numpy(pos).cuda(), torch.from_numpy(th).cuda(), n_rot, hd))
    finally:
        thi.thi_set_kernel_family(prev)
    assert np.isfinite(got.astype(np.float32)).all()
    rows = np.unique(np.concatenate([synth.sample_rows(53, M, 6), [0, 15, 16, 32, M - 1]]))
    y, s = oracle.rmsnorm_qkv_rope(x[rows], g, 1e-6, w, pos[rows], th, n_rot, hd)
    check(got[rows], y, s, "rmsnorm_qkv_rope", argmax=False)
