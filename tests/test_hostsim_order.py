"""The replay in the host build with the waves of a workgroup in drawn orders
(HIPSIM_ORDER): steps that only a barrier may order come in any order, so a
missing barrier shows as another result, an access out of bounds or a
deadlock.  The star schema and the S-largest input under all their plans."""
import os
import subprocess
import sys

import pytest

HOSTSIM = os.path.join(os.path.dirname(os.path.abspath(__file__)), "hostsim")


@pytest.mark.parametrize("seed", [1])
def test_replay_in_drawn_wave_orders(tmp_path_factory, seed):
    sys.path.insert(0, HOSTSIM)
    import build as hostsim_build
    built = hostsim_build.build(sanitize=True, jobs=8)
    data = tmp_path_factory.getbasetemp() / "hostsim_tiny"
    if not (data / "meta.txt").exists():
        subprocess.run([sys.executable, os.path.join(HOSTSIM, "make_inputs.py"), str(data), "--tiny"],
                       check=True, capture_output=True)
    r = subprocess.run([os.path.join(built, "replay"), str(data), "star", "slarge"], capture_output=True,
                       text=True, timeout=600, env=dict(os.environ, HIPSIM_ORDER=str(seed), HIPSIM_STEPS="1"))
    out = r.stdout + r.stderr
    assert r.returncode == 0 and "all checks passed" in out, out[-3000:]
