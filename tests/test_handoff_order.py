"""The hand-off between workgroups (handoff_last) as it is compiled for gfx950.

Pieces of a split bucket or range leave their rows in memory and the last one
reads them all, from another XCD's L2.  Before a workgroup takes its ticket
the device-scope release (buffer_wbl2) has to have been waited for; without
the wait the ticket can overtake the rows.  The order of instructions decides
that, so the test reads the assembly of the kernels that hand off (built here,
device code only; nothing runs)."""
import importlib.util
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1905_13376_amd")
SOURCES = {"linear": 10, "star": 2, "fm": 2}       # hand-offs of each file's kernels, merged forms included

ATOMIC = re.compile(r"^\s+(global|flat|buffer)_atomic_")
STORE = re.compile(r"^\s+(global|flat|buffer|scratch)_store_")
WAIT = re.compile(r"^\s+s_waitcnt\b.*vmcnt\(0\)")


def _builder():
    spec = importlib.util.spec_from_file_location("_mj_build", os.path.join(PKG, "build.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    b = _builder()
    out = tmp_path_factory.mktemp("asm")

    def cc(name):
        dst = str(out / (name + ".s"))
        cmd = [b.HIPCC] + b.FLAGS + ["--cuda-device-only", "-S", os.path.join(b.CSRC, name + ".hip"), "-o", dst]
        r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, r.stderr[-3000:]
        return name, open(dst).read().splitlines()

    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        return dict(ex.map(cc, SOURCES))


def _handoffs(lines):
    """(line of the write-back, waited before the next atomic, waited before the barrier) of every release that
    is followed by an atomic: the fences of other kinds (a threadfence before a barrier) have none."""
    found = []
    for i, ln in enumerate(lines):
        if not ln.strip().startswith("buffer_wbl2 sc1"):
            continue
        after = False
        j = i + 1
        while j < len(lines) and not ATOMIC.match(lines[j]) and "s_barrier" not in lines[j]:
            after = after or bool(WAIT.match(lines[j]))
            j += 1
        if j == len(lines) or "s_barrier" in lines[j]:
            continue
        k = i - 1                                   # back to the barrier, then to the waves' own wait
        while "s_barrier" not in lines[k]:
            k -= 1
        k -= 1
        while not WAIT.match(lines[k]) and not STORE.match(lines[k]):
            k -= 1
        found.append((i + 1, after, bool(WAIT.match(lines[k]))))
    return found


@pytest.mark.parametrize("name", sorted(SOURCES))
def test_write_back_is_waited_for_before_the_ticket(assembly, name):
    found = _handoffs(assembly[name])
    assert len(found) == SOURCES[name], found
    assert all(after for _, after, _ in found), f"{name}: a ticket is taken before the write-back is done: {found}"
    assert all(before for _, _, before in found), f"{name}: a store may follow the waves' wait: {found}"
