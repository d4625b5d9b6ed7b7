"""Hashed joins and cascades in workspaces without room for the tables' narrow
forms (as sized for a plan of other tables): the same counts, down to the
sizes that are refused."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, fixed_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("algo", ["3WAY", "CASCADE"])
@pytest.mark.parametrize("nb", [6, 9, 10])
def test_smaller_workspaces(algo, nb):
    import torch
    import paper_1905_13376_amd as mj
    ctx = mj.Context()
    rng = np.random.default_rng(nb)
    n, dom = 20000, 9000
    R, S, T = (rng.integers(0, dom, size=(n, 2)).astype(np.uint32) for _ in range(3))
    Rd, Sd, Td = dev(R), dev(S), dev(T)
    want = oracle.linear3_count(R, S, T, dom)
    p = fixed_plan(mj, ctx, mj.LINEAR, Rd, Sd, Td, dom, algo=getattr(mj, "ALGO_" + algo), log2_nb=nb, log2_nc=nb,
                   seed=0x99, flags=mj.PLAN_NO_DENSE)
    buf = torch.empty(p.workspace_bytes, dtype=torch.uint8, device="cuda")
    size, least = p.workspace_bytes, 0
    while size > 4096:
        ws = buf[:size]
        try:
            if algo == "3WAY":
                got = ctx.linear3_count(Rd, Sd, Td, dom, plan=p, workspace=ws)
            else:
                got = ctx.cascade2_count(mj.LINEAR, Rd, Sd, Td, dom, plan=p, workspace=ws)
        except mj.MJError as e:
            assert "WORKSPACE" in str(e)
            break
        np.testing.assert_array_equal(mj.as_u64(got), want)
        least, size = size, int(size * 0.9)
    assert 0 < least < 5 << 20                       # the narrow forms alone take 16 MiB at 9 bits
    ctx.close()
