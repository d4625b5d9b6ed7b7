"""Which dense linear joins run without a partition: one rule for the planner's
estimate and for the call.  Its line is 40,960 tuples a relation, whatever the
A domain up to 2^24; beyond that the tables are not direct-indexed and the
planner must not count on them.  Counts equal the oracle's on both sides."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mj():
    import paper_1905_13376_amd as mj
    return mj


def _run(mj, n_r, n_s, a_domain):
    rng = np.random.default_rng(n_r + n_s)
    R = np.stack([rng.integers(0, a_domain, n_r), rng.integers(0, 4096, n_r)], 1).astype(np.uint32)
    S = rng.integers(0, 4096, (n_s, 2)).astype(np.uint32)
    ctx = mj.Context()
    Rd, Sd = dev(R), dev(S)
    p = ctx.plan(mj.LINEAR, Rd, Sd, Sd, a_domain)
    assert p.flags & mj.PLAN_DENSE_KEYS
    est = p.est_ms_3way
    p.algo = mj.ALGO_3WAY
    ctx.profile(True)
    ctx.profile_read()
    got = mj.as_u64(ctx.linear3_count(Rd, Sd, Sd, a_domain, plan=p))
    names = {k.split(":")[-1] for k in ctx.profile_read()}
    ctx.profile(False)
    ctx.close()
    np.testing.assert_array_equal(got, oracle.linear3_count(R, S, S, a_domain))
    return names, est


@pytest.mark.parametrize("n_r,n_s,a_domain,small", [
    (40960, 40960, 4096, True), (1000, 40960, 1 << 24, True), (40960, 1000, 1 << 24, True),
    (40961, 1000, 4096, False), (1000, 40961, 4096, False), (49152, 49152, 4096, False)])
def test_line(mj, n_r, n_s, a_domain, small):
    names, est = _run(mj, n_r, n_s, a_domain)
    assert ("k_small_count" in names) == small, names
    assert ("k_range_count" in names) != small, names
    assert (est < 0.05) == small, est                 # three launches, or the partitioned join's model


def test_estimate_beyond_the_direct_indexed_domain(mj):
    names, est = _run(mj, 3000, 3000, (1 << 24) + 1)
    assert "k_small_count" not in names, names
    assert est > 0.05, est
