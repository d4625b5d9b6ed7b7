"""The table builds' hand-off in the host build (tests/hostsim/handoff_check.cpp):
the last piece of a split bucket meets other pieces' counts and rows as they
were before the kernel, and under AddressSanitizer no access leaves a buffer."""
import os
import subprocess
import sys

HOSTSIM = os.path.join(os.path.dirname(os.path.abspath(__file__)), "hostsim")


def test_late_rows_stay_inside_the_buffers():
    sys.path.insert(0, HOSTSIM)
    import build as hostsim_build
    exe = os.path.join(hostsim_build.build(sanitize=True, jobs=8), "handoff_check")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "all checks passed" in r.stdout, (r.stdout + r.stderr)[-3000:]
