"""Grids of the row kernels at the largest admitted numbers of (layer, head)
pairs, without a device: tests/native/launch_driver.cpp replaces the HIP launch
entry points, calls pack and unpack (per token, per variant, grouped) and checks
that every launch stays below 2^32 threads, that the launches of a kernel
together cover every chunk once and that the shortest requests get no workgroups
without a token."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_row_launches_stay_below_the_grid_limit(tmp_path):
    from paper_2606_08635_amd import build as B

    if not os.path.exists(B.HIPCC):
        pytest.skip("hipcc not found")
    objs = [os.path.join(B.BUILD_DIR, os.path.splitext(s)[0] + ".o") for s in B.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        B.build()
    exe = str(tmp_path / "launches")
    drv = os.path.join(ROOT, "tests", "native", "launch_driver.cpp")
    r = subprocess.run([B.HIPCC, *B.FLAGS, "-c", drv, "-o", exe + ".o"], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([B.HIPCC, "--offload-arch=gfx950", "-o", exe, exe + ".o", *objs], capture_output=True, text=True,
                       timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr[-2000:]
