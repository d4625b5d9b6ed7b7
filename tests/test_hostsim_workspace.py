"""Planned workspaces of small linear joins in the host build
(tests/hostsim/workspace_check.cpp): no room for narrow tables that the plan's
route does not read, and the autotuner's candidates still run in them."""
import os
import subprocess
import sys

HOSTSIM = os.path.join(os.path.dirname(os.path.abspath(__file__)), "hostsim")


def test_small_plans_ask_for_little():
    sys.path.insert(0, HOSTSIM)
    import build as hostsim_build
    exe = os.path.join(hostsim_build.build(sanitize=True, jobs=8), "workspace_check")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "all checks passed" in r.stdout, (r.stdout + r.stderr)[-3000:]
