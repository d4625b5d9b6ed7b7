"""Heavy work items of the cyclic join in the host build
(tests/hostsim/heavy_check.cpp): a join value with 2^27 tuples on both sides
has 2^32 items, which neither wrap to none nor stop the queue's counter."""
import os
import subprocess
import sys

HOSTSIM = os.path.join(os.path.dirname(os.path.abspath(__file__)), "hostsim")


def test_items_beyond_32_bits():
    sys.path.insert(0, HOSTSIM)
    import build as hostsim_build
    exe = os.path.join(hostsim_build.build(sanitize=True, jobs=8), "heavy_check")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "all checks passed" in r.stdout, (r.stdout + r.stderr)[-3000:]
