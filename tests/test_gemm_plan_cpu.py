"""Which GEMM configuration csrc/plan.hip picks, asked on the CPU (256 compute units): the picks where a price had been wrong, and
that the shapes of the GPU tests run the kernels they are listed for."""
import os
import shutil
import subprocess
from collections import namedtuple

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")

PLAIN, GATE_UP = 0, 2
Plan = namedtuple("Plan", "config tiles grid cut parts rows ranges per spread helpers")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_driver")
    res = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Wno-unused-command-line-argument", "-o", exe,
                          os.path.join(ROOT, "paper_2605_25655_amd", "csrc", "plan.hip"),
                          "-x", "hip", os.path.join(ROOT, "tests", "plan", "plan_driver.cpp")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]

    def ask(epilogue, M, N, K):
        out = subprocess.run([exe], input=f"{epilogue} {M} {N} {K}\n", capture_output=True, text=True, check=True).stdout.split()
        return Plan(out[0], *map(int, out[1:]))
    return ask


# A share of a tile pays a workgroup's fixed time in full, and so do the few-token configurations: with both left out, these ran the
# configuration in the last column (times in microseconds there and here).
@pytest.mark.parametrize("epilogue,M,N,K,config,was", [
    (PLAIN, 129, 4096, 11008, "DEEP", "TALL"),          # 41.5 -> 36.6
    (PLAIN, 203, 4096, 11008, "DEEP", "TALL"),          # 42.4 -> 38.7
    (PLAIN, 82, 332, 792, "MID", "FEW128"),             # 12.3 -> 8.4
    (PLAIN, 123, 124, 7440, "MID", "FEW128"),           # 32.5 -> 7.6
    (PLAIN, 96, 1536, 512, "MID", "FEW128"),
    (GATE_UP, 50, 25832, 176, "SMALL", "FEW128"),       # 11.6 -> 9.1
    (GATE_UP, 97, 7648, 104, "FEW128", None),           # the few-token kernel 7.1, here 6.0
    (PLAIN, 61, 28750, 640, "FEW64", None),             # 12.9, here 11.4
    (PLAIN, 72, 12288, 4096, "MID", None),
    (PLAIN, 512, 8192, 8192, "DEEP", None),
    (GATE_UP, 219, 312, 2304, "FEW128", "TALL"),        # 24.8 -> 19.8
    (PLAIN, 153, 4474, 6400, "FEW128", "TALL"),         # 39.2 -> 30.4
    (PLAIN, 606, 3961, 5024, "DEEP", "SMALL"),          # 52.0 -> 41.2
])
def test_picks(plan, epilogue, M, N, K, config, was):
    assert plan(epilogue, M, N, K).config == config


def test_tiles_of_256_tokens_are_not_cut_for_a_tenth_of_a_microsecond(plan):
    assert plan(GATE_UP, 204, 12936, 9856)[:4] == ("ONE", 203, 203, 0)      # all cut 172, whole 144


def _cut(p):
    how = "whole" if p.cut == 0 else "shares" if p.parts == 0 else "ranges"
    return "rounds + " + how if 0 < p.cut < p.tiles else how


def test_the_gpu_tests_run_the_kernels_they_are_listed_for(plan):
    from tests.test_parity_gpu import FEW_KERNEL, KERNELS, RAGGED, ROW_TILES
    for kind, M, N, K, config, cut in KERNELS:
        p = plan(GATE_UP if kind == "G" else PLAIN, M, N, K)
        assert (p.config, _cut(p)) == (config, cut), (kind, M, N, K, p)
    both = [(e, M, N if e == PLAIN else N // 2 // 8 * 8, K) for e in (PLAIN, GATE_UP) for M, N, K in FEW_KERNEL]
    few = [plan(*shape) for shape in both]
    assert all(p.config == "MID" for p in few), [(s, p) for s, p in zip(both, few) if p.config != "MID"]
    for e in (PLAIN, GATE_UP):      # every height of tile for every token tile that has it, shared and alone where it is built for both
        seen = {(p.rows, 64 if s[1] <= 64 else 96 if s[1] <= 96 else 128) for s, p in zip(both, few) if s[0] == e}
        assert {(32, 64), (144, 64), (112, 64), (112, 96), (96, 64), (96, 96), (80, 64), (80, 96), (80, 128), (64, 64), (64, 128), (48, 96),
                (32, 96), (32, 128)} <= seen, seen
        assert {(32, True), (32, False), (80, True), (80, False)} <= {(p.rows, p.ranges > 1) for s, p in zip(both, few) if s[0] == e}
    for e in (PLAIN, GATE_UP):
        shapes = [(M, N if e == PLAIN else N // 2 // 8 * 8, K) for M, N, K in ROW_TILES]
        assert [plan(e, *t).config for t in shapes] == ["R224", "R224", "R192", "R192", "R160", "R160", "R160"]
    assert {plan(PLAIN, *t).config for t in RAGGED} == {"MID", "DEEP", "SMALL"}


def test_the_gpu_tests_of_spread_starts_and_of_decode_sizes(plan):
    import paper_2605_25655_amd as thi
    from tests.test_parity_gpu import DECODE_WORKSPACE, FEW_DECODE, SPREAD_STARTS
    picks = [plan(PLAIN, *t) for t in SPREAD_STARTS]      # two token tiles, stages of 64 k
    assert all(p.config == "FEW128" and 128 < t[0] <= 256 and t[2] % 64 == 0 for t, p in zip(SPREAD_STARTS, picks)), picks
    assert {_cut(p) for p in picks} == {"whole", "ranges"} and any(p.helpers for p in picks)
    few = [plan(PLAIN, *t) for t in FEW_DECODE]
    assert all(p.config == "MID" for p in few), few
    assert {p.rows for p in few if p.ranges == 1} == {32, 48, 64, 80, 96, 112, 128, 144, 176}
    assert {p.rows for p in few if p.ranges > 1} >= {32, 48, 64, 80, 96, 112, 128}
    assert {p.rows for t, p in zip(FEW_DECODE, few) if p.ranges > 1 and p.spread and t[2] % 128} >= {48, 96, 112, 128}
    assert {48, 96} <= {p.rows for p in few if p.ranges > 1 and not p.spread}
    assert any(p.per < p.rows for p in few) and any(p.per % 16 for p in few)
    kinds = {"P": (PLAIN, 0), "Q": (PLAIN, 1), "G": (GATE_UP, 2)}
    seen = {k: set() for k in kinds}
    for kind, M, N, K in DECODE_WORKSPACE:
        epilogue, fused = kinds[kind]
        p = plan(epilogue, M, N, K)
        assert p.config == "MID" and p.ranges > 1 and thi.thi_query_kernel_family(M, N, K, fused) == 2, (kind, M, N, K, p)
        seen[kind].add((p.rows, p.spread))
    assert seen["Q"] >= {(32, 0), (32, 1), (48, 1), (96, 1), (112, 1)} and seen["P"] >= {(48, 0), (64, 1), (112, 0)} and len(seen["G"]) == 3, seen


def test_whole_128_tiles_leave_units_that_touch_the_weights(plan):
    from tests.test_parity_gpu import TOUCHED
    picks = [plan(PLAIN, *t) for t in TOUCHED]
    assert all(p.config in ("DEEP", "FEW128") and p.cut == 0 and 8 <= p.tiles == p.grid <= 256 - 48 for p in picks), picks
    assert all(p.helpers > 0 and p.helpers % 8 == 0 and p.grid + p.helpers <= 256 for p in picks), picks
    assert {p.config for p in picks} == {"DEEP", "FEW128"} and {8, 208} <= {p.tiles for p in picks}
    # two token tiles whose starts are spread over k, gate/up, and few tiles with a long K: not these
    assert plan(PLAIN, 203, 12288, 4096).tiles == 192 and plan(PLAIN, 203, 4096, 4096).cut == 64
    assert plan(PLAIN, 372, 512, 4096).cut > 0


def test_rows_beyond_31_bits_do_not_wrap(plan):
    """More virtual rows than an int holds: no tile count of the few-token kernel comes near the compute units'."""
    assert plan(GATE_UP, 40, 2 ** 30 + 8, 8).config != "MID"
    import paper_2605_25655_amd as thi
    assert thi.thi_query_kernel_family(40, 2 ** 30 + 8, 8, 2) == 1      # the stream-K kernel, which takes any number of rows


@pytest.mark.parametrize("M,N,K,fused,family", [(1, 4096, 512, 0, 3), (32, 20480, 512, 0, 3), (32, 20481, 512, 0, 1), (16, 16384, 264, 1, 3),
                                                (16, 16400, 264, 1, 1), (8, 16384, 256, 0, 3), (8, 16400, 256, 0, 1),
                                                (8, 4096, 128, 2, 3), (8, 4104, 128, 2, 1), (8, 10240, 264, 2, 3), (8, 10248, 264, 2, 1)])
def test_small_k_is_reported_as_it_runs(M, N, K, fused, family):
    import paper_2605_25655_amd as thi
    assert thi.thi_query_kernel_family(M, N, K, fused) == family
    for forced in (1, 3, 4):
        prev = thi.thi_set_kernel_family(forced)
        try:
            assert thi.thi_query_kernel_family(M, N, K, fused) == 1
        finally:
            thi.thi_set_kernel_family(prev)


def test_rows_longer_than_the_gemm_addresses():
    """256 rows of more than 2^23 values lie further apart than 32 bits of bytes: the stream-K kernel takes them."""
    import paper_2605_25655_amd as thi
    for M, N, K in ((40, 200, 2 ** 23 + 8), (129, 8, 2 ** 24 + 2 ** 17 + 8), (300, 2048, 2 ** 23 + 64)):
        for forced in (0, 2):
            prev = thi.thi_set_kernel_family(forced)
            try:
                assert thi.thi_query_kernel_family(M, N, K, 0) == 1
                assert forced == 0 or thi.thi_query_kernel_family(M, N, 2 ** 23, 0) == 2
            finally:
                thi.thi_set_kernel_family(prev)


def test_the_single_launch_mlp_is_planned_once_and_where_it_exists(tmp_path):
    """Outside 17..32 tokens an MLP call plans its two projections and nothing else; inside it asks once whether one launch would serve."""
    exe = str(tmp_path / "host_calls")
    csrc = os.path.join(ROOT, "paper_2605_25655_amd", "csrc")
    res = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Wno-unused-command-line-argument",
                          "-Wl,--wrap=_ZN3thi17rowblock_split_okEiiiii", "-o", exe, os.path.join(csrc, "api.hip"), os.path.join(csrc, "plan.hip"),
                          "-x", "hip", os.path.join(ROOT, "tests", "sanitize", "api_stubs.cpp"), os.path.join(ROOT, "tests", "plan", "host_calls.cpp")],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]

    def tried(M, H, I):
        out = subprocess.run([exe], input=f"{M} {H} {I}\n", capture_output=True, text=True, check=True).stdout.split()
        return tuple(map(int, out))
    for H, I in ((512, 1376), (4096, 11008), (5120, 13824), (8192, 28672)):
        for M in (1, 8, 16, 33, 64, 200):
            mlp, gate_up, down = tried(M, H, I)
            assert gate_up == 0 and mlp == down, (M, H, I, mlp, gate_up, down)
    mlp, gate_up, down = tried(32, 4096, 11008)      # the one shape that is fused: the question, then the split that its launch takes
    assert 0 < gate_up and mlp <= gate_up + 4, (mlp, gate_up, down)


def test_a_forced_row_block_split_leaves_the_other_kernels_alone():
    """It says how row blocks are shared: where they would run they do, and the few-token kernel stays where it stands for the stream-K kernel."""
    import paper_2605_25655_amd as thi
    shapes = [(M, N, K, f) for M in (1, 5, 16, 32) for N, K in ((300, 5000), (1000, 2048), (5120, 8200), (8192, 8192), (13824, 5120), (36000, 1040)) for f in (0, 1, 2)]
    prev_family = thi.thi_set_kernel_family(0)
    prev = thi.thi_set_rowblock_split(0)
    try:
        free = {s: thi.thi_query_kernel_family(*s) for s in shapes}
        thi.thi_set_rowblock_split(1)
        single = {s: thi.thi_query_kernel_family(*s) for s in shapes}
    finally:
        thi.thi_set_rowblock_split(prev)
        thi.thi_set_kernel_family(prev_family)
    assert not [s for s in shapes if free[s] == 2 and single[s] == 1], [(s, single[s]) for s in shapes if free[s] == 2]
    assert any(free[s] == 2 == single[s] for s in shapes) and any(free[s] == 2 and single[s] == 4 for s in shapes)
