"""What the few-token kernel does in front of its first load, when nothing is in flight yet: as many instructions as it takes, counted in the library as
built, and quotients that are products."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
OBJDUMP = os.environ.get("LLVM_OBJDUMP", "/opt/rocm/llvm/bin/llvm-objdump")


def _setup(tmp_path):
    """For each of its kernels: the instructions up to the first load, and the loads that stand in front of the first barrier."""
    from paper_2605_25655_amd import build
    lib = shutil.copy(build.LIB, str(tmp_path / "lib.so"))
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    counts, loads, ahead = {}, {}, True
    for code in sorted(str(p) for p in tmp_path.iterdir() if p.name.endswith("gfx950")):
        if "gemm_midI" not in subprocess.run([OBJDUMP, "-t", code], capture_output=True, text=True, check=True).stdout:
            continue
        kernel, n = None, 0
        for line in subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", code], capture_output=True, text=True, check=True).stdout.split("\n"):
            label = re.match(r"^(?:[0-9a-f]+ )?<(\S+)>:", line)
            if label:
                m = re.search(r"gemm_midILi(\d+)ELi(\d+)ELi(\d+)ELb(\d)E", label.group(1))
                kernel, n, ahead = (tuple(map(int, m.groups())), 0, True) if m else (None, 0, True)
            elif kernel and line.strip():
                n += 1
                if "global_load_lds" in line:
                    counts.setdefault(kernel, n)
                    loads[kernel] = loads.get(kernel, 0) + ahead
                ahead = ahead and "s_barrier" not in line
    return counts, loads


@pytest.mark.skipif(shutil.which(OBJDUMP) is None, reason="llvm-objdump not found")
def test_little_stands_in_front_of_the_first_load(tmp_path):
    counts, loads = _setup(tmp_path)
    assert len(counts) > 90, len(counts)
    # one and a half times what the kernels of 32 rows and 32 tokens have as built, and for the tallest (176 rows of gate/up pairs, eight loads a wave) a little
    # more than they have; setting up each load by itself took 463 and 865
    assert counts[32, 32, 0, 0] <= 276, counts[32, 32, 0, 0]
    assert max(counts.values()) <= 600, max(counts.items(), key=lambda c: c[1])
    # 32 rows and 64 tokens: six stages of two or three loads in both loops, the first of them with and without the non-temporal hint; a branch for
    # the last k-tile of a ragged K made them 63
    assert loads[32, 64, 0, 0] <= 42, loads[32, 64, 0, 0]


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")
def test_quotients_are_exact(tmp_path):
    exe = str(tmp_path / "quotient")
    res = subprocess.run([HIPCC, "-O2", "-std=c++17", "--offload-arch=gfx950", "-Wno-unused-command-line-argument", "-o", exe, "-x", "hip",
                          os.path.join(ROOT, "tests", "plan", "quotient_driver.cpp")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
