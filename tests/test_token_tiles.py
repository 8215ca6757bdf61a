"""Above 128 tokens: the few-token kernel with several token tiles.  On the CPU: what csrc/plan.hip deals covers the product, one round of
workgroups, tiles that the kernel is built for.  On the GPU: results against the oracle at the edges of its tiles."""
import os
import random
import shutil
import subprocess

import numpy as np
import pytest

from paper_2605_25655_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
PLAIN, GATE_UP = 0, 2

# Two token tiles of each height (64..128) with one token more and less, three to eight of them; outputs that fill no tile and end inside a
# quad, tiles of 32..144 rows, alone and shared; K of one k-tile, ragged, with fewer k-tiles than stages, rows of 4 KiB (spread starts).
SHAPES = [
    (129, 1000, 1096), (137, 510, 72), (150, 4096, 4096), (192, 2003, 2048), (193, 1536, 520), (200, 851, 1560), (208, 6001, 2056), (224, 4096, 1032),
    (225, 3001, 904), (256, 512, 1376), (257, 339, 3672), (301, 2810, 1296), (552, 580, 6568), (640, 801, 544), (160, 5120, 5128), (150, 7000, 10248),
    (206, 5969, 4256), (209, 2482, 4856), (232, 1995, 6144), (574, 542, 5200), (640, 2322, 3368), (349, 5428, 4776), (201, 10944, 5384),
]


def _driver(tmp_path, *flags, source="token_tiles_driver.cpp"):
    exe = str(tmp_path / "driver")
    res = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Wno-unused-command-line-argument", *flags, "-o", exe,
                          os.path.join(ROOT, "paper_2605_25655_amd", "csrc", "plan.hip"), "-x", "hip",
                          os.path.join(ROOT, "tests", "plan", source)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    return exe


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")
def test_a_call_plans_the_gemm_once(tmp_path):
    exe = _driver(tmp_path, "-Xarch_host", "-finstrument-functions")
    calls = [(PLAIN, *s) for s in SHAPES] + [(PLAIN, 203, 12288, 4096), (PLAIN, 512, 5120, 13824), (PLAIN, 2048, 8192, 8192), (GATE_UP, 150, 2816, 1024)]
    text = "".join("%d %d %d %d\n" % c for c in calls)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    lines = [line for line in out if line]
    assert len(lines) == len(calls) + 1 and int(lines[-1]) == len(calls), lines[-1]


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")
def test_only_weights_that_one_workgroup_reads_pass_the_caches(tmp_path):
    exe = _driver(tmp_path, source="load_hints_driver.cpp")
    rng = random.Random(5)
    calls = [(PLAIN, *s) for s in SHAPES] + [(GATE_UP, 72, 11008, 4096), (PLAIN, 72, 12288, 4096), (GATE_UP, 256, 1376, 512)]
    calls += [(rng.choice([PLAIN, GATE_UP]), rng.randint(1, 432), rng.randint(8, 13000), 8 * rng.randint(8, 1600)) for _ in range(4000)]
    text = "".join("%d %d %d %d\n" % c for c in calls)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    lines = [tuple(map(int, line.split())) for line in out if line]
    assert len(lines) == len(calls)
    seen = set()
    for call, (weights, tiles_m, *waves) in zip(calls, lines):
        for w, bits in enumerate(waves):
            for i in range(32):      # load i of wave w is number w + 8 i of the k-tile
                assert bool(bits >> i & 1) == (w + 8 * i < weights and tiles_m == 1), (call, weights, tiles_m, w, i)
        seen.add((weights > 0, weights % 8 != 0, tiles_m > 1))
    assert seen >= {(True, True, False), (True, False, False), (True, True, True), (True, False, True)}, seen


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")
def test_plans_cover_the_product_in_one_round(tmp_path):
    exe = _driver(tmp_path)
    rng = random.Random(3)
    calls = [(PLAIN, *s) for s in SHAPES]
    calls += [(rng.choice([PLAIN, GATE_UP]), rng.randint(100, 1100), 8 * rng.randint(1, 1600), 8 * rng.randint(1, 3200)) for _ in range(4000)]
    text = "".join("%d %d %d %d\n" % c for c in calls)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    plans = [tuple(map(int, line.split())) for line in out if line]
    assert len(plans) == len(calls)
    built = {64: {32, 48, 64, 80, 96, 112, 144}, 96: {32, 48, 64, 80, 96, 112}, 112: {64, 96}, 128: {32, 48, 64, 80}}
    seen = set()
    for i, ((e, M, N, K), (rows, tiles, ranges, per, tiles_m, per_m)) in enumerate(zip(calls, plans)):
        if rows == 0:
            continue
        tall = 64 if per_m <= 64 else 96 if per_m <= 96 else 112 if per_m <= 112 and rows in (64, 96) else 128
        assert M > 128 and per_m % 4 == 0 and per_m <= 128 and (tiles_m - 1) * per_m < M <= tiles_m * per_m, (e, M, N, K)
        assert per % 4 == 0 and per * (2 if e == GATE_UP else 1) <= rows and rows in built[tall], (e, M, N, K)
        tiles_n = tiles // tiles_m
        assert tiles == tiles_n * tiles_m and (tiles_n - 1) * per < N <= tiles_n * per, (e, M, N, K)
        assert tiles * ranges <= 256 and ranges <= (K + 127) // 128, (e, M, N, K)
        if i < len(SHAPES):
            seen.add((tall, ranges > 1))
    assert all(p[0] for p in plans[:len(SHAPES)]), [s for s, p in zip(SHAPES, plans) if not p[0]]
    assert seen >= {(tall, shared) for tall in (64, 96, 112, 128) for shared in (False, True)}, seen
    assert {p[0] for p in plans[:len(SHAPES)]} >= {32, 48, 64, 80, 96, 112} and any(p[3] < p[0] for p in plans[:len(SHAPES)])


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_several_token_tiles(M, N, K):
    import torch

    import oracle
    import paper_2605_25655_amd as thi
    from tests.gpu_common import Runner, to_dev, to_host
    from tests.parity import check
    print(f"[case] token tiles M={M} N={N} K={K}", flush=True)
    x, w, g = synth.random_problem(12000 + M + N + K, M, N, K)
    rng = np.random.Generator(np.random.Philox(key=12100 + M + N + K))
    res = rng.standard_normal((M, N)).astype(np.float16)
    hd, I = 8, N // 16 * 8
    n_rot = N // hd // 2 * hd
    pos = rng.integers(0, 4096, size=M).astype(np.int32)
    th = (10000.0 ** (-np.arange(0, hd, 2, dtype=np.float64) / hd)).astype(np.float32)
    rows = np.unique(np.concatenate([synth.sample_rows(41, M, 8), [0, M // 2 - 1, M // 2, M - 1]]))
    r = Runner(M, K, max(I, K), N)
    xd, wd, gd, rd = to_dev(x), to_dev(w), to_dev(g), to_dev(res)
    a = [to_host(r.linear_residual(xd, wd, rd)) for _ in range(3)]
    assert all(np.array_equal(a[0].view(np.uint16), v.view(np.uint16)) for v in a[1:]), "not reproducible"
    y, s = oracle.linear_residual(x[rows], w, res[rows])
    check(a[0][rows], y, s, "linear + residual", argmax=False)
    c = to_host(r.rmsnorm_qkv_rope(xd, gd, 1e-6, wd, torch.from_numpy(pos).cuda(), torch.from_numpy(th).cuda(), n_rot, hd))
    y, s = oracle.rmsnorm_qkv_rope(x[rows], g, 1e-6, w, pos[rows], th, n_rot, hd)
    check(c[rows], y, s, "rmsnorm_qkv_rope", argmax=False)
    outs = [a[0], c]
    if I:
        h = to_host(r.swiglu_gate_up(xd, wd[:I], wd[I:2 * I]))
        y, s = oracle.swiglu_gate_up(x[rows], w[:I], w[I:2 * I])
        check(h[rows], y, s, "gate/up", argmax=False)
        outs.append(h)
    # every output was written: the GEMM's own kernels, forced, agree on all of them to fp16's rounding of two sums in another order
    prev = thi.thi_set_kernel_family(2)
    try:
        ref = [to_host(r.linear_residual(xd, wd, rd)), to_host(r.rmsnorm_qkv_rope(xd, gd, 1e-6, wd, torch.from_numpy(pos).cuda(), torch.from_numpy(th).cuda(), n_rot, hd))]
        if I:
            ref.append(to_host(r.swiglu_gate_up(xd, wd[:I], wd[I:2 * I])))
    finally:
        thi.thi_set_kernel_family(prev)
    for got, want in zip(outs, ref):
        got, want = got.astype(np.float32), want.astype(np.float32)
        # each rounds its sum once (half a unit in the last place, 2^-11, so 2^-10 between them), and the fp32 sums differ by a few of their
        # own units (2^-24 of the sum of the products' magnitudes, here below K times the largest result) where a result cancels
        bound = np.maximum(np.abs(got), np.abs(want)) * 2.0 ** -10 + 2.0 ** -24 * K * max(1.0, float(np.abs(want).max()))
        assert (np.abs(got - want) <= bound).all()


# Gate/up pairs alone: the highest tile, 144 rows, which the plain kind reaches nowhere
TALLEST = (293, 3440, 3960)


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")
def test_gate_up_halves_and_the_highest_tile_are_token_tiles_too(tmp_path):
    exe = _driver(tmp_path)
    calls = [(GATE_UP, M, N // 16 * 8, K) for M, N, K in SHAPES] + [(GATE_UP, *TALLEST)]
    text = "".join("%d %d %d %d\n" % c for c in calls)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    plans = [tuple(map(int, line.split())) for line in out if line]
    assert len(plans) == len(calls) and all(p[0] for p in plans), [c for c, p in zip(calls, plans) if not p[0]]
    assert {p[0] for p in plans[:-1]} >= {32, 48, 64, 80, 96, 112} and plans[-1][0] == 144, plans


@pytest.mark.gpu
def test_gate_up_of_the_highest_tile():
    import oracle
    from tests.gpu_common import Runner, to_dev, to_host
    from tests.parity import check
    M, I, K = TALLEST
    print(f"[case] token tiles of 144 rows, gate/up M={M} I={I} K={K}", flush=True)
    x, w, _ = synth.random_problem(17000, M, 2 * I, K)
    rows = np.unique(np.concatenate([synth.sample_rows(71, M, 8), [0, 59, 60, M - 1]]))
    r = Runner(M, K, I, K)
    xd, wd = to_dev(x), to_dev(w)
    h = [to_host(r.swiglu_gate_up(xd, wd[:I], wd[I:])) for _ in range(3)]
    assert all(np.array_equal(h[0].view(np.uint16), v.view(np.uint16)) for v in h[1:]), "not reproducible"
    assert np.isfinite(h[0].astype(np.float32)).all()
    y, s = oracle.swiglu_gate_up(x[rows], w[:I], w[I:])
    check(h[0][rows], y, s, "gate/up", argmax=False)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(129, 1000, 1096), (150, 4096, 4096), (200, 851, 1560), (257, 339, 3672), (640, 2322, 3368)])
def test_residual_in_place_over_several_token_tiles(M, N, K):
    from tests.gpu_common import Runner, to_dev, to_host
    print(f"[case] token tiles, residual in place M={M} N={N} K={K}", flush=True)
    x, w, _ = synth.random_problem(17100 + M + N + K, M, N, K)
    res = np.random.Generator(np.random.Philox(key=17200 + M + N + K)).standard_normal((M, N)).astype(np.float16)
    r = Runner(M, K, K, N)
    xd, wd, rd = to_dev(x), to_dev(w), to_dev(res)
    apart = to_host(r.linear_residual(xd, wd, rd))
    assert np.isfinite(apart.astype(np.float32)).all()
    for _ in range(3):
        assert np.array_equal(apart.view(np.uint16), to_host(r.linear_residual(xd, wd, rd, in_place=True)).view(np.uint16))


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")
def test_only_tiles_that_a_plan_can_ask_for_are_built():
    import re

    from paper_2605_25655_amd import build
    with open(build.LIB, "rb") as f:
        names = set(re.findall(rb"gemm_midILi(\d+)ELi(\d+)E", f.read()))
    heights = {}
    for rows, tall in names:
        heights.setdefault(int(tall), set()).add(int(rows))
    assert heights == {32: {32, 48, 64, 80, 96, 112, 128, 144, 176}, 64: {32, 48, 64, 80, 96, 112, 144}, 96: {32, 48, 64, 80, 96, 112},
                       112: {64, 96}, 128: {32, 48, 64, 80}}, heights
