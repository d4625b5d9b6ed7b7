"""Dense keys: the small joins (no partition, at most 49,152 tuples a
relation), the packed 4-byte range pairs and the unpacked ones, at the edges
of their sizes, domains, layouts and shared partitions.  Counts are integers
and must equal the oracle's; a bound broken after planning gives all ones."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu
ONES = np.uint64(2 ** 64 - 1)


@pytest.fixture(scope="module")
def mj():
    import paper_1905_13376_amd as mj
    return mj


def _columns(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a.view(np.int32).T)).to("cuda").t()


def _odd(a):
    """Rows at an address that is not 16-byte aligned, four words apart."""
    import torch
    buf = torch.zeros(a.shape[0] * 4 + 8, dtype=torch.int32, device="cuda")
    v = buf[2:2 + 4 * a.shape[0]].view(-1, 4)[:, :2]
    v.copy_(torch.from_numpy(a.view(np.int32)))
    return v


def _rel(rng, n, d0, d1, hub):
    r = np.stack([rng.integers(0, d0, size=n), rng.integers(0, d1, size=n)], 1).astype(np.uint32)
    if hub:
        r[: n // 3, 0] = d0 - 1                       # a crowded range: split into pieces
    r[-1] = (d0 - 1, d1 - 1)
    return r


@pytest.mark.parametrize("nr,ns,nt,da,db,dc", [
    (1, 1, 1, 1, 1, 1), (2, 63, 8191, 5, 64, 65), (8192, 8193, 16385, 4096, 4097, 4095),
    (49152, 49151, 49152, 65536, 3000, 100000), (49153, 49152, 2, 64, 4096, 4097),
    (131071, 131072, 131073, 8191, 8192, 8193), (140000, 60001, 200003, 300000, 120000, 400000),
    (600001, 70001, 50001, 1 << 20, 1000, 131071)])
@pytest.mark.parametrize("layout", ["rows", "columns", "odd"])
@pytest.mark.parametrize("hub", [False, True])
def test_dense_sizes_domains_layouts(mj, nr, ns, nt, da, db, dc, layout, hub):
    rng = np.random.default_rng(nr + 3 * ns + 7 * nt)
    R, S, T = _rel(rng, nr, da, db, hub), _rel(rng, ns, db, dc, hub), _rel(rng, nt, dc, 9, hub)
    ctx = mj.Context()
    put = {"rows": dev, "columns": _columns, "odd": _odd}[layout]
    Rd, Sd, Td = put(R), put(S), put(T)
    p = ctx.plan(mj.LINEAR, Rd, Sd, Td, da)
    p.algo = mj.ALGO_3WAY
    got = mj.as_u64(ctx.linear3_count(Rd, Sd, Td, da, plan=p))
    np.testing.assert_array_equal(got, oracle.linear3_count(R, S, T, da))
    ctx.close()


@pytest.mark.parametrize("n", [3000, 60000, 300000])
@pytest.mark.parametrize("a_domain", [4096, 5000, 1 << 17])
def test_shared_partition_with_other_bounds(mj, n, a_domain):
    """R = S = T as one tensor whose first column stays below 4000 and whose
    second below 4096: one partition held to all three bounds."""
    rng = np.random.default_rng(n)
    F = np.stack([rng.integers(0, 4000, size=n), rng.integers(0, 4096, size=n)], 1).astype(np.uint32)
    ctx = mj.Context()
    Fd = dev(F)
    p = ctx.plan(mj.LINEAR, Fd, Fd, Fd, a_domain)
    assert p.flags & mj.PLAN_DENSE_KEYS
    p.algo = mj.ALGO_3WAY
    np.testing.assert_array_equal(mj.as_u64(ctx.linear3_count(Fd, Fd, Fd, a_domain, plan=p)),
                                  oracle.linear3_count(F, F, F, a_domain))
    ctx.close()


@pytest.mark.parametrize("n", [20000, 60000, 300000])
@pytest.mark.parametrize("what", ["R.a", "R.b", "S.b", "S.c", "T.c"])
def test_bound_broken_after_planning(mj, n, what):
    """A key at or past its bound: all ones where the key indexes a sum, no
    match where it is only looked up."""
    rng = np.random.default_rng(n)
    R, S, T = (rng.integers(0, 4096, size=(n, 2)).astype(np.uint32) for _ in range(3))
    for X in (R, S, T):
        X[0] = 4095
    ctx = mj.Context()
    for bad in (4096, 4097, 1 << 20, 0xFFFFFFFF):
        Rd, Sd, Td = dev(R), dev(S), dev(T)
        p = ctx.plan(mj.LINEAR, Rd, Sd, Td, 4096)
        p.algo = mj.ALGO_3WAY
        X, col = {"R.a": (Rd, 0), "R.b": (Rd, 1), "S.b": (Sd, 0), "S.c": (Sd, 1), "T.c": (Td, 0)}[what]
        X[n // 2, col] = bad - (1 << 32) if bad >= 1 << 31 else bad
        got = mj.as_u64(ctx.linear3_count(Rd, Sd, Td, 4096, plan=p))
        if what in ("R.b", "S.c"):
            R2, S2 = Rd.cpu().numpy().view(np.uint32), Sd.cpu().numpy().view(np.uint32)
            np.testing.assert_array_equal(got, oracle.linear3_count(R2, S2, T, 4096))
        else:
            assert (got == ONES).all()
    ctx.close()


@pytest.mark.parametrize("pad", [0, 60000])
def test_sums_past_the_narrow_copies(mj, pad):
    """deg past 16 bits, W at and past the saturating copy and past 32 bits;
    `pad` more tuples of other keys take the join past the small sizes."""
    def rows(x, y):
        return np.stack(np.broadcast_arrays(np.asarray(x), np.asarray(y)), 1).astype(np.uint32)
    ws = [65534, 65535, 65536, 1, 700]
    S = np.concatenate([rows(np.full(min(w, 40000) if not pad else w, b), 0) for b, w in enumerate(ws)] +
                       [rows(np.full(30000, 9), 1), rows(np.arange(pad) % 50 + 20, 5)])
    T = np.concatenate([rows([0], 9), rows(np.full(40000 if not pad else 70000, 1), 9)])
    R = np.concatenate([rows(np.arange(20) % 7, np.arange(20) % 10), rows(np.arange(pad) % 3000, 9)])
    if not pad:
        S = S[:49152]
    ctx = mj.Context()
    Rd, Sd, Td = dev(R), dev(S), dev(T)
    p = ctx.plan(mj.LINEAR, Rd, Sd, Td, 3000)
    assert p.flags & mj.PLAN_DENSE_KEYS
    p.algo = mj.ALGO_3WAY
    np.testing.assert_array_equal(mj.as_u64(ctx.linear3_count(Rd, Sd, Td, 3000, plan=p)),
                                  oracle.linear3_count(R, S, T, 3000))
    ctx.close()
