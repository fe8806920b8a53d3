"""What the library's calls launch, on the CPU: a driver in tests/host/ stands
in for the HIP runtime and carries out what the kernels do to the control
block, so that a launch or a copy can be made to fail in the middle of a call
and launch shapes can be read.  No GPU is used."""
import os
import shutil
import subprocess

import pytest

import paper_1903_09043_amd as A

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    A.lib()
    exe = str(tmp_path_factory.mktemp("host") / "launch_driver")
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
           os.path.join(ROOT, "tests", "host", "launch_driver.cpp"), "-x", "none", A.LIB_PATH,
           "-Wl,-rpath," + os.path.dirname(A.LIB_PATH), "-rdynamic", "-ldl", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.mark.parametrize("what", ["failed_step", "batch_tiling", "shares", "placement", "one_wave", "tuned_2d"])
def test_launches(driver, what, tmp_path):
    """failed_step: the time steps after a call that ended in an error are
    those of the new call's own states.  batch_tiling: ars_batch_get_tiling
    reports what is launched and bound.  shares: the schedule of a march's
    (tile, plane) pairs takes every pair once and its longest share is no
    longer than that of an even split.  placement: neighbouring shares meet on
    one XCD whatever the number of workgroups.  one_wave: 2D steps that can
    give every SIMD at most one workgroup do.  tuned_2d: tuning keeps the
    untuned launch of a 2D step where that is the fastest."""
    r = subprocess.run([driver, what, str(tmp_path / "tune.txt")], capture_output=True, text=True, timeout=120)
    print(r.stdout[-4000:], r.stderr[-2000:])
    assert r.returncode == 0 and r.stdout.strip().endswith("ok")
