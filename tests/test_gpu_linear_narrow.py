"""Hashed tables with their narrow form (9 or 10 bucket bits) and without it:
values at the narrow slots' limit, the key 0xFFFFFFFF, few and many keys a
bucket (full tables, spills, moved entries), heavy keys built in pieces.
Counts are integers and must equal the oracle's."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, fixed_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mj():
    import paper_1905_13376_amd as mj
    return mj


def _keys(rng, distinct):
    k = rng.integers(0, 1 << 32, size=distinct, dtype=np.uint64).astype(np.uint32)
    k[0] = 0xFFFFFFFF
    k[-1] = 0
    return k


def _check(mj, R, S, T, a_domain, nb, nc, cascade):
    ctx = mj.Context()
    Rd, Sd, Td = dev(R), dev(S), dev(T)
    want = oracle.linear3_count(R, S, T, a_domain)
    p = fixed_plan(mj, ctx, mj.LINEAR, Rd, Sd, Td, a_domain, log2_nb=nb, log2_nc=nc, seed=0x1234 + nb,
                   flags=mj.PLAN_NO_DENSE)
    np.testing.assert_array_equal(mj.as_u64(ctx.linear3_count(Rd, Sd, Td, a_domain, plan=p)), want)
    if cascade:
        q = fixed_plan(mj, ctx, mj.LINEAR, Rd, Sd, Td, a_domain, algo=mj.ALGO_CASCADE, log2_nb=nb, log2_nc=nc,
                       seed=0x77, flags=mj.PLAN_NO_DENSE)
        np.testing.assert_array_equal(mj.as_u64(ctx.cascade2_count(mj.LINEAR, Rd, Sd, Td, a_domain, plan=q)), want)
    ctx.close()


@pytest.mark.parametrize("nb,nc", [(8, 9), (9, 10), (10, 9), (10, 10), (11, 8)])
@pytest.mark.parametrize("distinct,n", [(40, 20003), (1000, 60003), (60000, 200003), (400000, 300007)])
def test_keys_per_bucket(mj, nb, nc, distinct, n):
    rng = np.random.default_rng(nb * 100 + nc + distinct)
    b, c = _keys(rng, distinct), _keys(rng, distinct)
    R = np.stack([rng.integers(0, 5000, size=n), b[rng.integers(0, distinct, size=n)]], 1).astype(np.uint32)
    S = np.stack([b[rng.integers(0, distinct, size=n)], c[rng.integers(0, distinct, size=n)]], 1).astype(np.uint32)
    T = np.stack([c[rng.integers(0, distinct, size=n)], rng.integers(0, 9, size=n)], 1).astype(np.uint32)
    _check(mj, R, S, T, 5000, nb, nc, distinct >= 1000)


@pytest.mark.parametrize("nb,nc", [(9, 9), (10, 10), (2, 12)])
@pytest.mark.parametrize("hub", [0, 30000, 120000])
def test_values_at_the_narrow_limit(mj, nb, nc, hub):
    """Multiplicities and sums of 16382, 16383, 16384 and beyond 32 bits' half,
    beside small ones and a hub built in pieces."""
    rng = np.random.default_rng(nb + hub)
    b, c = _keys(rng, 3000), _keys(rng, 3000)
    mult = [16382, 16383, 16384, 70000, 1, 2]
    T = np.concatenate([np.stack([np.full(m, c[i + 5]), np.arange(m)], 1) for i, m in enumerate(mult)] +
                       [np.stack([c, c], 1)] + ([np.stack([np.full(hub, c[0]), np.arange(hub)], 1)] if hub else []))
    S = np.concatenate([np.stack([b, c], 1), np.stack([b[rng.integers(0, 3000, 40000)], c[rng.integers(0, 3000, 40000)]], 1),
                        np.stack([np.full(16382, b[50]), np.full(16382, c[60])], 1),
                        np.stack([np.full(16383, b[51]), np.full(16383, c[61])], 1)] +
                       ([np.stack([np.full(hub, b[7]), c[rng.integers(0, 3000, hub)]], 1)] if hub else []))
    R = np.stack([rng.integers(0, 700, 50000), b[rng.integers(0, 3000, 50000)]], 1)
    if hub:
        R = np.concatenate([R, np.stack([np.full(hub, 699), b[rng.integers(0, 3000, hub)]], 1)])
    R, S, T = (np.ascontiguousarray(x.astype(np.uint32)) for x in (R, S, T))
    _check(mj, R, S, T, 700, nb, nc, hub == 0)
