"""The pinned result slots of sampling calls, on the CPU with a stand-in for the
HIP runtime's calls (tests/sanitize/host_slots_main.cpp): a call that fails on a
captured stream leaves no slot taken."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_captured_calls_leave_no_slot_taken(tmp_path):
    import paper_1902_00530_amd as L
    exe = str(tmp_path / "host_slots")
    lib = os.path.dirname(L.LIB_PATH)
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-o", exe,
                    os.path.join(ROOT, "tests", "sanitize", "host_slots_main.cpp"), "-L" + lib, "-llbm",
                    "-Wl,-rpath," + lib, "-Wl,-rpath,/opt/rocm/lib", "-Wl,-rpath-link,/opt/rocm/lib"], check=True,
                   capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "host slots: ok" in r.stdout, r.stdout[:2000] + r.stderr
