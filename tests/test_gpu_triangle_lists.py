"""The cyclic join's staged lists at the edges of their sizes: lists staged by
a wave (at most 448 entries) or by a workgroup (slices of at most 2048), lists
streamed by a lane (at most 16) or by the wave in pieces of 64, groups around
a wave's chunk, bags (repeated tuples), every share.  Totals are integers and
must equal the oracle's."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, fixed_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mj():
    import paper_1905_13376_amd as mj
    return mj


def _hub(rng, x, y, g, bag):
    """One hub B value with x R tuples (`bag` of each A value, if set), g S tuples (its C values, plus one
    small group), each C value with y T tuples; half of T's A values are R's."""
    a = rng.permutation(1 << 20)[:max(x, 1)].astype(np.uint32)
    if bag:
        a = a[rng.integers(0, max(1, x // bag), size=x)]
    R = np.stack([a[:x], np.full(x, 7, np.uint32)], axis=1)
    c = rng.integers(0, max(1, min(g, 40)), size=g).astype(np.uint32) + 100
    S = np.stack([np.full(g, 7, np.uint32), c], axis=1)
    S = np.concatenate([S, np.array([[9, 100], [7, 0xFFFFFFFF]], np.uint32)])
    cs = np.unique(S[:, 1])
    T = []
    for v in cs:
        t = rng.integers(0, 1 << 20, size=y).astype(np.uint32)
        hit = rng.random(y) < 0.5
        t[hit] = a[rng.integers(0, a.size, size=int(hit.sum()))]
        T.append(np.stack([np.full(y, v, np.uint32), t], axis=1))
    T = np.concatenate(T)
    R = np.concatenate([R, np.array([[a[0], 9], [0xFFFFFFFF, 7]], np.uint32)])
    T = np.concatenate([T, np.array([[100, 0xFFFFFFFF]], np.uint32)])
    return R.astype(np.uint32), S.astype(np.uint32), T.astype(np.uint32)


@pytest.mark.parametrize("x,y,g", [
    (1, 1, 1), (15, 16, 63), (17, 15, 64), (64, 17, 65), (65, 63, 129), (128, 64, 31), (447, 65, 257), (448, 447, 300), (449, 448, 65),
    (511, 510, 70), (512, 511, 64), (513, 300, 64), (1024, 513, 4095), (4094, 257, 4097), (2047, 1025, 90), (2048, 64, 2049), (2049, 17, 2048),
    (4096, 5, 700), (4097, 16, 513), (8193, 4097, 40), (20000, 1500, 8200)])
@pytest.mark.parametrize("bag", [0, 3, 200])
def test_staged_and_streamed_list_sizes(mj, x, y, g, bag):
    rng = np.random.default_rng(x * 7 + y * 3 + g + bag)
    R, S, T = _hub(rng, x, y, g, bag)
    want = oracle.triangle3_count(R, S, T)
    ctx = mj.Context()
    Rd, Sd, Td = dev(R), dev(S), dev(T)
    for share in (0, 2, 5):
        p = fixed_plan(mj, ctx, mj.TRIANGLE, Rd, Sd, Td, algo=mj.ALGO_3WAY, log2_share=share, seed=11 + share)
        assert int(mj.as_u64(ctx.triangle3_count(Rd, Sd, Td, plan=p))[0]) == want, share
    ctx.close()


@pytest.mark.parametrize("nr,ns,nt", [
    (1, 16384, 16385), (16385, 4097, 131073), (131073, 131072, 20479), (4096, 300000, 20481), (262145, 3, 16383)])
def test_sorts_of_different_sizes_together(mj, nr, ns, nt):
    """The four key arrays of one join, some sorted in one workgroup, some in
    passes whose scatter adds up the histogram rows, some with scanned rows;
    with the materialised join for the order inside equal keys (stability)."""
    rng = np.random.default_rng(nr + ns + nt)
    R, S, T = (rng.integers(0, 2500, size=(n, 2)).astype(np.uint32) for n in (nr, ns, nt))
    R[0] = S[0] = T[0] = (0xFFFFFFFF, 0xFFFFFFFF)
    ctx = mj.Context()
    Rd, Sd, Td = dev(R), dev(S), dev(T)
    p = fixed_plan(mj, ctx, mj.TRIANGLE, Rd, Sd, Td, algo=mj.ALGO_3WAY, seed=5)
    assert int(mj.as_u64(ctx.triangle3_count(Rd, Sd, Td, plan=p))[0]) == oracle.triangle3_count(R, S, T)
    import torch
    out = torch.zeros((5000, 4), dtype=torch.int32, device="cuda")
    got, total = ctx.linear3_materialize(Rd, Sd, Td, first=7, out=out)
    want = np.asarray(oracle.linear3_materialize(R, S, T, 7, 5000)[0], dtype=np.uint32).reshape(-1, 4)
    assert np.array_equal(got.cpu().numpy().view(np.uint32)[:want.shape[0]], want)
    ctx.close()
