"""The planner's column maxima (one launch over all key columns) and |R |x| S|
at the edges of the kernels' rounds: the largest value first, last or in the
middle, sizes around a wave, a workgroup and a workgroup's round of four."""
import numpy as np
import pytest

from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mj():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1905_13376_amd as m
    return m


@pytest.mark.parametrize("n", [1, 63, 65, 256, 1023, 1025, 4097, 600_001])
def test_plan_maxima_and_join_size(mj, n):
    ctx = mj.Context()
    g = np.random.default_rng(n)
    for at in sorted({0, n // 2, n - 1}):
        R, S, T = (g.integers(0, 50, size=(n, 2)).astype(np.int32) for _ in range(3))
        R[at] = (60, 61)
        S[at] = (62, 63)
        T[at, 0] = 64
        Rd, Sd, Td = dev(R), dev(S), dev(T)
        p = ctx.plan(mj.LINEAR, Rd, Sd, Td, 61)
        assert p.flags & mj.PLAN_DENSE_KEYS
        assert (p.b_domain, p.c_domain) == (63, 65)
        want = int((np.bincount(R[:, 1], minlength=64).astype(np.int64)
                    * np.bincount(S[:, 0], minlength=64)).sum())
        assert p.join2_size == want == ctx.join2_size(Rd, Sd)
        with pytest.raises(mj.MJError) as e:
            ctx.plan(mj.LINEAR, Rd, Sd, Td, 60)
        assert e.value.status == -2
    ctx.close()
