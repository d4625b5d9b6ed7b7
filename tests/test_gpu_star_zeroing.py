"""The star join's per-A counts start from zero whoever clears them: few of
them the workgroups of the pass over S, many (beside a small S, which gets few
workgroups) a launch of their own.  Counts equal the oracle's, and a large A
domain costs about what writing it takes."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mj():
    import paper_1905_13376_amd as mj
    return mj


def _join(n_s, a_domain):
    rng = np.random.default_rng(n_s + a_domain)
    keys = rng.choice(1 << 30, 4096, replace=False)
    R = np.stack([rng.integers(0, a_domain, 4096), keys], 1).astype(np.uint32)
    S = np.stack([rng.choice(keys, n_s), rng.integers(0, 4096, n_s)], 1).astype(np.uint32)
    T = rng.integers(0, 4096, (4096, 2)).astype(np.uint32)
    return R, S, T


# one and two workgroups, at and just above the entries they zero themselves
@pytest.mark.parametrize("n_s,a_domain", [(100, 1), (16384, 1 << 15), (16384, (1 << 15) + 1), (16385, 1 << 16),
                                          (16385, (1 << 16) + 1), (5000, 1 << 22)])
def test_counts_on_a_buffer_with_old_values(mj, n_s, a_domain):
    import torch
    R, S, T = _join(n_s, a_domain)
    ctx = mj.Context()
    Rd, Sd, Td = dev(R), dev(S), dev(T)
    p = ctx.plan(mj.LINEAR, Rd, Sd, Td, a_domain)
    p.algo = mj.ALGO_STAR
    out = torch.full((a_domain,), -7, dtype=torch.int64, device="cuda")
    got = mj.as_u64(ctx.linear3_count(Rd, Sd, Td, a_domain, plan=p, out=out))
    np.testing.assert_array_equal(got, oracle.linear3_count(R, S, T, a_domain))
    ctx.close()


def test_a_large_domain_costs_its_writing(mj):
    import torch

    def us(fn, n=10):
        fn()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        for _ in range(n):
            fn()
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) / n * 1e3

    ctx = mj.Context()
    t = {}
    for a_domain in (1 << 10, 1 << 24):
        Rd, Sd, Td = (dev(x) for x in _join(4096, a_domain))
        p = ctx.plan(mj.LINEAR, Rd, Sd, Td, a_domain)
        p.algo = mj.ALGO_STAR
        ws = torch.empty(p.workspace_bytes, dtype=torch.uint8, device="cuda")
        out = torch.empty(a_domain, dtype=torch.int64, device="cuda")
        t[a_domain] = us(lambda: ctx.linear3_count(Rd, Sd, Td, a_domain, plan=p, out=out, workspace=ws))
    fill = us(lambda: out.zero_())
    # one workgroup clearing them all took 70 times the fill
    assert t[1 << 24] - t[1 << 10] < 10 * fill, (t, fill)
    ctx.close()
