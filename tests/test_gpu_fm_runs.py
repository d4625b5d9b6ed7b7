"""Distinct counts whose runs of T and S have lengths around the limits of
the sketch kernels (16 lanes a run up to 64 elements, waves of 512 elements
beyond), whose A values fill one range beyond a workgroup's share, whose
directory has long gaps, and where S and T are one relation.  Sketches must
equal the oracle's bit for bit, the estimates exactly."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1905_13376_amd as mj
    c = mj.Context()
    yield c
    c.close()


def _check(ctx, R, S, T, a_domain, seed, Sd=None, Td=None):
    Sd = dev(S) if Sd is None else Sd
    sk, est = ctx.linear3_distinct(dev(R), Sd, dev(T) if Td is None else Td, a_domain, seed=seed)
    a = np.unique(R[:, 0])
    al, want, want_est, _ = oracle.linear3_distinct(R, S, T, a, seed)
    sk = sk.cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(sk[al], want)
    np.testing.assert_array_equal(est.cpu().numpy()[al], want_est)
    absent = np.setdiff1d(np.arange(a_domain), al)
    assert not sk[absent].any()


def _runs(rng, lens, values):
    """(key, value) rows: key i has lens[i] rows, in any order."""
    k = np.repeat(np.arange(len(lens)), lens)
    return rng.permutation(np.stack([k, values(k.size)], 1)).astype(np.uint32)


@pytest.mark.parametrize("a_domain", [200, 70000, 1 << 19])
@pytest.mark.parametrize("longest", [64, 65, 511, 513, 1025, 7000])
def test_run_lengths(ctx, longest, a_domain):
    rng = np.random.default_rng(longest + a_domain)
    short = [1, 2, 15, 16, 17, 33]
    t_lens = short * 30 + [longest]
    T = _runs(rng, t_lens, lambda n: rng.integers(0, 1 << 32, n, dtype=np.uint64))
    s_lens = short * 20 + [64, longest, longest + 1]
    S = _runs(rng, s_lens, lambda n: rng.integers(0, len(short) * 30, n))
    S = np.concatenate([S, [[len(s_lens) - 1, len(t_lens) - 1], [7, len(t_lens) - 1]]]).astype(np.uint32)
    R = np.stack([rng.integers(0, a_domain, 3000), rng.integers(0, len(s_lens), 3000)], 1)
    hub = np.stack([np.full(9001, a_domain // 2), rng.integers(0, 40, 9001)], 1)   # one A value: split ranges
    R = np.concatenate([R[:50], hub, R[50:]]).astype(np.uint32)
    _check(ctx, R, S, T, a_domain, seed=longest)


@pytest.mark.parametrize("n,dom", [(1, 1), (63, 5), (4097, 3), (30000, 20000)])
def test_one_relation(ctx, n, dom):
    # S and T the same tensor, then equal ones
    rng = np.random.default_rng(n)
    F = rng.integers(0, dom, size=(n, 2)).astype(np.uint32)
    R = np.stack([rng.integers(0, 50, 60), rng.integers(0, dom, 60)], 1).astype(np.uint32)
    if n == 4097:
        R = R[:3]
    Fd = dev(F)
    _check(ctx, R, F, F, 50, 5, Fd, Fd)
    _check(ctx, R, F, F, 50, 5)
