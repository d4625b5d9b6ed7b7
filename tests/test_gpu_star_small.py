"""Star joins whose dimension tables every workgroup builds in LDS: sizes at
the limit of 4096 tuples and just above it, keys that share a bucket and a
slot, the key 0xFFFFFFFF, heavy keys, columns that are not packed, an A value
out of range.  Counts are integers and must equal the oracle's."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, fixed_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mj():
    import paper_1905_13376_amd as mj
    return mj


def _colliding(n):
    """Keys whose hashes share the top 11 bits in large groups and, in fours, the slot bits too."""
    i = np.arange(n, dtype=np.uint64)
    x, f = i % 4, i // 4                      # bits 19 and 20 of the hash; what the four share
    top, low = f % 97, f // 97
    h = (top << np.uint64(21)) | (x << np.uint64(19)) | ((low ^ x) & np.uint64(0x1FFF))
    inv = pow(0x9E3779B1, -1, 1 << 32)
    return ((h * np.uint64(inv)) & np.uint64(0xFFFFFFFF)).astype(np.uint32)


def _keys(rng, kind, n):
    if kind == "colliding":
        return _colliding(n)
    if kind == "dense":
        return np.arange(n, dtype=np.uint32)
    k = rng.integers(0, 1 << 32, size=n, dtype=np.uint64).astype(np.uint32)
    k[0] = 0xFFFFFFFF
    return k


def _rel(rng, lo, hi):
    return np.stack([lo, hi], 1).astype(np.uint32)


def _run(mj, R, S, T, a_domain, then=None):
    ctx = mj.Context()
    p = fixed_plan(mj, ctx, mj.LINEAR, R, S, T, a_domain, algo=mj.ALGO_STAR, seed=0x51)
    if then:
        then()
    got = mj.as_u64(ctx.linear3_count(R, S, T, a_domain, plan=p))
    ctx.close()
    return got


@pytest.mark.parametrize("kind", ["random", "dense", "colliding"])
@pytest.mark.parametrize("n_r,n_t", [(1, 1), (64, 65), (4095, 4096), (4096, 1000), (4097, 4096), (4096, 4097)])
def test_sizes_and_keys(mj, kind, n_r, n_t):
    rng = np.random.default_rng(n_r + 3 * n_t)
    kb, kc = _keys(rng, kind, n_r), _keys(rng, kind, n_t)
    n_s = 3 * 16384 + 8191
    R = _rel(rng, rng.integers(0, 700, n_r), rng.permutation(kb))
    S = _rel(rng, kb[rng.integers(0, n_r, n_s)], kc[rng.integers(0, n_t, n_s)])
    S[::7, 0] = rng.integers(0, 1 << 32, size=len(S[::7]), dtype=np.uint64)
    S[3::11, 1] = 0xFFFFFFFF
    T = _rel(rng, kc[rng.integers(0, n_t, n_t)], rng.integers(0, 9, n_t))
    np.testing.assert_array_equal(_run(mj, dev(R), dev(S), dev(T), 700), oracle.linear3_count(R, S, T, 700))


@pytest.mark.parametrize("n_s", [1, 2, 8191, 8193, 40001])
def test_heavy_keys_and_plain_columns(mj, n_s):
    # every key of T the same, a few keys of R; S in columns of its own, then
    # rows that start 8 bytes off 16-byte alignment
    rng = np.random.default_rng(n_s)
    R = _rel(rng, rng.integers(0, 50, 4096), rng.integers(0, 3, 4096))
    S = _rel(rng, rng.integers(0, 4, n_s), rng.integers(0, 2, n_s))
    T = _rel(rng, np.zeros(4096), rng.integers(0, 9, 4096))
    want = oracle.linear3_count(R, S, T, 50)
    Rd, Td = dev(R), dev(T)
    Sd = dev(S).t().contiguous().t()
    np.testing.assert_array_equal(_run(mj, Rd, Sd, Td, 50), want)
    off = dev(np.concatenate([S[:1], S]))[1:]
    np.testing.assert_array_equal(_run(mj, Rd, off, Td, 50), want)


def test_a_value_out_of_range(mj):
    # written after planning: every count all ones if such a value joins
    R, S = np.array([[4, 7]], dtype=np.uint32), np.array([[7, 9]], dtype=np.uint32)
    for c, want in ((9, np.uint64(2**64 - 1)), (8, np.uint64(0))):
        Rd = dev(R)
        got = _run(mj, Rd, dev(S), dev(np.array([[c, 0]], dtype=np.uint32)), 5, lambda: Rd.add_(dev(np.array([[1, 0]], dtype=np.uint32))))
        assert (got == want).all()
