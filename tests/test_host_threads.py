"""Threads of the slot BP workgroups, no GPU: a compute unit holds 16 wavefronts of the kernel (128 registers,
four per SIMD), so the workgroups meant to share one have to fit in that."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_workgroups_of_a_tier_are_resident(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "threads_check")
    r = subprocess.run([hipcc, "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                        os.path.join(ROOT, "paper_2406_18655_amd", "csrc"),
                        os.path.join(HERE, "host", "threads_check.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    v = list(map(int, subprocess.run([exe], capture_output=True, text=True, timeout=60).stdout.split()))
    threads = dict(zip(v[::2], v[1::2]))
    assert all(t % 64 == 0 and 256 <= t <= 1024 for t in threads.values())
    assert all(wg * threads[wg] // 64 <= 16 for wg in (1, 2, 3, 4))
    # the tiers of decoder creation fill the compute unit
    assert [wg * threads[wg] // 64 for wg in (1, 2, 4)] == [16, 16, 16]
