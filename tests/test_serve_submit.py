"""vp_submit and vp_poll do not wait while the scheduler launches a job's kernels, and
jobs that end are seen between two launches (csrc/serve_core.cpp), on the CPU with an
executor whose launches take their time; plainly and with ThreadSanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2005_09316_amd", "csrc")


@pytest.mark.parametrize("sanitizer", [None, "thread"])
def test_callers_do_not_wait_for_launches(tmp_path, sanitizer):
    exe = str(tmp_path / "serve_submit_test")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-pthread", "-Wall", "-I" + CSRC, "-I" + os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "serve_submit_test.cpp"), os.path.join(CSRC, "serve_core.cpp"), "-o", exe]
    if sanitizer:
        cmd.insert(1, "-fsanitize=" + sanitizer)
    subprocess.run(cmd, check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, TSAN_OPTIONS="halt_on_error=1 second_deadlock_stack=1"))
    assert r.returncode == 0 and "PASS" in r.stdout, r.stdout + r.stderr
    assert "ThreadSanitizer" not in r.stderr, r.stderr
