"""Every launch's error reaches the caller (CPU: the HIP calls of the library are taken by
the driver `tests/sanitize/launch_main.cpp`, nothing is launched): along each branch of
every entry point's dispatch, any one failing launch must give MOE_ERR_DEVICE."""
import os
import shutil
import subprocess

import pytest

from paper_2607_08782_amd import moe

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_any_failing_launch_is_reported(tmp_path):
    if not os.path.exists(moe.LIB_PATH):
        from paper_2607_08782_amd import build
        build.build()
    exe = str(tmp_path / "launch_errors")
    # -rdynamic: the driver's definitions come before the runtime's
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "sanitize", "launch_main.cpp"), "-o", exe, "-ldl"],
                   check=True, timeout=120)
    r = subprocess.run([exe, moe.LIB_PATH], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "launch errors: OK" in r.stdout, r.stdout + r.stderr[-3000:]
