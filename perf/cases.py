"""Performance cases: the joins a program runs through the public entry points.

A case names a family, sizes and options; ``prepare`` draws the relations on
the GPU from the seed and makes what a program keeps between calls (the
context, the plan, the output buffer of a windowed result), ``run`` makes one
call.  The families and their ranges:

* ``linear``      R(A,B) |x| S(B,C) |x| T(C,D) counted per A, small dense ids
* ``hashed``      the same with keys spread over all 32-bit patterns
* ``adhoc``       the same without a plan at hand: planned inside the call
* ``cascade``     the same through the materialised binary cascade
* ``star``        a large fact relation between two small dimension relations
* ``distinct``    Flajolet-Martin distinct count of D per A
* ``materialize`` a window of the result tuples written out
* ``cyclic``      triangles: R(A,B) |x| S(B,C) |x| T(C,A)
* ``batch``       many joins of uneven size in one call
"""
import math

import numpy as np
import torch

import paper_1905_13376_amd as mj

DEV = "cuda"
M32 = 0xFFFFFFFF
FM_SEED = 0x9E3779B9


def listed():
    return [
        # the paper's uniform self-join at its small size: a call is latency and launches
        dict(name="linear_small", family="linear", dist="uniform", n_r=65536, n_s=65536, n_t=65536,
             domain=4096, cap=0, same=True, columns=False),
        # the benchmarked friends-of-friends-of-friends query: 2^24 edges, one relation three times
        dict(name="linear_powerlaw", family="linear", dist="powerlaw", n_r=1 << 24, n_s=1 << 24, n_t=1 << 24,
             domain=1 << 20, cap=4096, same=True, columns=False),
        # three relations of their own sizes whose keys are hashes (account numbers, not dense ids)
        dict(name="linear_hashed", family="hashed", dist="powerlaw", n_r=6000011, n_s=9999991, n_t=4194301,
             domain=524287, cap=65536, same=False, columns=False),
        # a question asked once over three column-stored tables of about a million rows
        dict(name="linear_adhoc", family="adhoc", dist="uniform", n_r=1200007, n_s=1999993, n_t=800011,
             domain=100003, cap=0, same=False, columns=True),
        # the binary cascade the paper compares against: |R |x| S| about 16 times an input
        dict(name="cascade", family="cascade", dist="powerlaw", n_r=1 << 20, n_s=1 << 20, n_t=1 << 20,
             domain=1 << 16, cap=4096, same=True, columns=False),
        # star schema: 2^26 facts, dimension relations that fit one workgroup
        dict(name="star_fact", family="star", n_r=4096, n_s=1 << 26, n_t=4096, a_domain=1024),
        # star schema whose dimension relations are too large for that (S the largest relation)
        dict(name="star_large_dims", family="star", n_r=65536, n_s=1 << 25, n_t=65536, a_domain=16384),
        # distinct friends of friends of friends per person, sketched
        dict(name="distinct", family="distinct", dist="powerlaw", n_r=1 << 22, n_s=1 << 22, n_t=1 << 22,
             domain=1 << 18, cap=4096, same=True, columns=False),
        # 2^25 result tuples of a self-join read out as one window
        dict(name="materialize", family="materialize", dist="powerlaw", n_r=1 << 20, n_s=1 << 20, n_t=1 << 20,
             domain=1 << 16, cap=4096, same=True, columns=False, first=12345, rows=1 << 25),
        # triangles of the R-MAT graph of scale 22 (2^27 directed tuples, one symmetric relation)
        dict(name="triangles_rmat22", family="cyclic", shape="rmat", scale=22, edges=1 << 26),
        # a cyclic join of three different skewed relations (no symmetry to use)
        dict(name="cyclic_general", family="cyclic", shape="three", n_r=1 << 20, n_s=1500007, n_t=999983,
             domain=65536),
        # a mixed batch of joins of 10^3 to 10^6 tuples, half linear and half cyclic
        dict(name="batch_64", family="batch", count=64, lo=3.0, hi=6.0, mix=4000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    f = rng.choice(["linear", "linear", "hashed", "adhoc", "cascade", "star", "distinct", "materialize", "cyclic",
                    "cyclic", "batch"])
    if f == "star":
        wide = rng.random() < 0.5
        n_r, n_t = ((_log(rng, 1 << 13, 1 << 18), _log(rng, 1 << 13, 1 << 18)) if wide
                    else (_log(rng, 64, 4096), _log(rng, 64, 4096)))
        return dict(family=f, n_r=n_r, n_s=_log(rng, 1 << 20, 1 << 25 if wide else 1 << 26), n_t=n_t,
                    a_domain=_log(rng, 16, 65536))
    if f == "cyclic":
        shape = rng.choice(["rmat", "three", "uniform"])
        if shape == "three":
            n = _log(rng, 2000, 1 << 21)
            return dict(family=f, shape=shape, n_r=n, n_s=max(1, int(n * rng.uniform(0.5, 1.5))),
                        n_t=max(1, int(n * rng.uniform(0.5, 1.5))), domain=max(64, int(n / rng.uniform(12, 20))))
        scale = rng.randint(10, 20)
        return dict(family=f, shape=shape, scale=scale, edges=max(64, int((1 << scale) * rng.uniform(4, 16))))
    if f == "batch":
        return dict(family=f, count=rng.randint(8, 64), lo=3.0, hi=round(rng.uniform(4.5, 6.0), 2),
                    mix=rng.randrange(1 << 30))
    top = {"linear": 1 << 24, "hashed": 1 << 23, "adhoc": 1 << 22, "cascade": 1 << 20, "distinct": 1 << 22,
           "materialize": 1 << 20}[f]
    same = rng.random() < 0.4
    n_r = _log(rng, 1000, top)
    n_s, n_t = (n_r, n_r) if same else [min(top, max(1, int(n_r * rng.uniform(0.4, 2.5)))) for _ in range(2)]
    case = dict(family=f, dist=rng.choice(["uniform", "powerlaw"]), n_r=n_r, n_s=n_s, n_t=n_t,
                domain=max(64, int(max(n_r, n_s, n_t) / rng.uniform(10, 24))), cap=rng.choice([4096, 65536, 0]),
                same=same, columns=rng.random() < 0.3)
    if f in ("cascade", "materialize"):
        case["cap"] = 4096                       # a hub's squared degree is not what is written out
    if f == "materialize":
        case["first"] = rng.choice([0, 1, 1009])
        case["rows"] = _log(rng, 1000, 1 << 25)
    return case


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _ints(g, hi, n):
    return torch.randint(0, hi, (n,), generator=g, device=DEV, dtype=torch.int64)


def _powerlaw(g, n, m, cap):
    """m directed edges over n vertices: capped rank-Zipf(1.1) out-degrees,
    destinations by the copy model of preferential attachment."""
    cap = min(cap, m) if cap else m
    base = torch.arange(1, n + 1, dtype=torch.float64, device=DEV) ** -1.1
    hi = 1.0
    limit = float(max(cap, (m + n - 1) // n))
    while float(torch.clamp(hi * base, max=limit).sum()) < m and hi < 1e18:
        hi *= 2.0
    lo = 0.0
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        if float(torch.clamp(mid * base, max=limit).sum()) < m:
            lo = mid
        else:
            hi = mid
    deg = torch.clamp(hi * base, max=limit).floor().to(torch.int64)
    src = torch.repeat_interleave(torch.randperm(n, generator=g, device=DEV), deg)[:m]
    src = torch.cat([src, _ints(g, n, m - src.numel())])            # the fractions' remainder, uniform
    src = src[torch.randperm(m, generator=g, device=DEV)]
    e = torch.arange(m, device=DEV)
    own = torch.rand(m, generator=g, device=DEV) < 0.5
    prev = (torch.rand(m, generator=g, device=DEV, dtype=torch.float64) * e.clamp(min=1)).to(torch.int64)
    parent = torch.where(own | (e == 0), e, torch.minimum(prev, (e - 1).clamp(min=0)))
    for _ in range(40):                                             # pointer doubling: 2^40 hops
        nxt = parent[parent]
        if torch.equal(nxt, parent):
            break
        parent = nxt
    return src, _ints(g, n, m)[parent]


def _pairs(g, case, n):
    d = case["domain"]
    if case["dist"] == "powerlaw":
        return _powerlaw(g, d, n, case["cap"])
    return _ints(g, d, n), _ints(g, d, n)


def _rel(x, y, columns=False):
    """An [n, 2] int32 relation: rows, or two columns seen as rows."""
    if columns:
        return torch.stack([x, y]).to(torch.int32).t()
    return torch.stack([x, y], dim=1).to(torch.int32)


def _scramble(x):
    """Small ids to 32-bit patterns (an odd multiple modulo 2^32: one to one), as int32 values."""
    y = (x * 0x9E3779B1 + 0x7F4A7C15) & M32
    return torch.where(y >= 1 << 31, y - (1 << 32), y)


def _symmetric(g, n, lo, hi):
    """Distinct undirected edges as both directed tuples, ids relabelled, shuffled."""
    ok = lo != hi
    key = torch.unique((torch.minimum(lo, hi)[ok] << 32) | torch.maximum(lo, hi)[ok])
    perm = torch.randperm(n, generator=g, device=DEV)
    x, y = perm[key >> 32], perm[key & M32]
    order = torch.randperm(2 * key.numel(), generator=g, device=DEV)
    return _rel(torch.cat([x, y])[order], torch.cat([y, x])[order])


def _rmat(g, scale, edges):
    u = torch.zeros(edges, dtype=torch.int64, device=DEV)
    v = torch.zeros(edges, dtype=torch.int64, device=DEV)
    for _ in range(scale):                                          # quadrants .57 .19 .19 .05
        r = torch.rand(edges, generator=g, device=DEV)
        b, c = (r >= 0.57) & (r < 0.76), (r >= 0.76) & (r < 0.95)
        d = r >= 0.95
        u = (u << 1) | (c | d)
        v = (v << 1) | (b | d)
    return _symmetric(g, 1 << scale, u, v)


def _zipf_ids(g, n, m):
    """m vertex ids drawn with capped Zipf(1.1) weights."""
    w = torch.clamp(torch.arange(1, n + 1, dtype=torch.float64, device=DEV) ** -1.1 * n, max=float(min(4096, n - 1)))
    cdf = torch.cumsum(w / w.sum(), 0)
    i = torch.searchsorted(cdf, torch.rand(m, generator=g, device=DEV, dtype=torch.float64)).clamp(max=n - 1)
    return torch.randperm(n, generator=g, device=DEV)[i]


def _relations(case, seed):
    """R, S, T and the length of the per-A output."""
    g = _gen(seed)
    f = case["family"]
    if f == "star":
        keys = torch.unique(_ints(g, 1 << 31, 2 * case["n_r"] + 64))
        keys = keys[torch.randperm(keys.numel(), generator=g, device=DEV)][:case["n_r"]]
        R = _rel(_ints(g, case["a_domain"], keys.numel()), keys)
        T = _rel(_ints(g, case["n_t"], case["n_t"]), _ints(g, 1 << 31, case["n_t"]))
        n = case["n_s"]
        hit = torch.rand(n, generator=g, device=DEV) < 15.0 / 16.0
        b = torch.where(hit, keys[_ints(g, keys.numel(), n)], _ints(g, 1 << 31, n))
        return R, _rel(b, _ints(g, case["n_t"], n)), T, case["a_domain"]
    if f == "cyclic":
        if case["shape"] == "three":
            d = case["domain"]
            rels = []
            for n in (case["n_r"], case["n_s"], case["n_t"]):
                rels.append(_rel(_zipf_ids(g, d, n), _zipf_ids(g, d, n)))
            return rels[0], rels[1], rels[2], 0
        n, m = 1 << case["scale"], case["edges"]
        E = _rmat(g, case["scale"], m) if case["shape"] == "rmat" else _symmetric(g, n, _ints(g, n, m), _ints(g, n, m))
        return E, E, E, 0
    rels = []
    for n in (case["n_r"], case["n_s"], case["n_t"]):
        if rels and case["same"]:
            rels.append(rels[0])
            continue
        x, y = _pairs(g, case, n)
        if f == "hashed":                        # A stays an output index; B and C become 32-bit patterns
            k = len(rels)
            x = x if k == 0 else _scramble(x)
            y = y if k == 2 else _scramble(y)
        rels.append(_rel(x, y, case["columns"]))
    R, S, T = rels
    if f == "hashed" and case["same"]:
        S = _rel(_scramble(R[:, 0].long()), R[:, 1].long(), case["columns"])
        T = S
    return R, S, T, case["domain"]


def _batch_relations(case, seed):
    sizes = np.random.default_rng(case["mix"]).uniform(case["lo"], case["hi"], case["count"])
    joins = []
    for k in range(case["count"]):
        g = _gen(seed * 4096 + k)
        m = int(round(10 ** sizes[k]))
        n = max(64, m // 16)
        if k < case["count"] // 2:
            x, y = _powerlaw(g, n, m, 4096) if k % 2 else (_ints(g, n, m), _ints(g, n, m))
            F = _rel(x, y)
            joins.append((mj.LINEAR, F, F, F, n))
        else:
            if k % 2:
                E = _symmetric(g, n, _zipf_ids(g, n, m), _zipf_ids(g, n, m))
            else:
                E = _symmetric(g, n, _ints(g, n, m), _ints(g, n, m))
            joins.append((mj.TRIANGLE, E, E, E, 0))
    return joins


# ------------------------------------------------------------------ the calls
def prepare(case, seed):
    ctx = mj.Context()
    f = case["family"]
    if f == "batch":
        return dict(family=f, batch=ctx.batch(_batch_relations(case, seed)))
    R, S, T, a_domain = _relations(case, seed)
    st = dict(family=f, ctx=ctx, R=R, S=S, T=T, a_domain=a_domain)
    if f == "materialize":
        st["first"] = case["first"]
        st["out"] = torch.zeros((case["rows"], 4), dtype=torch.int32, device=DEV)
    elif f == "cyclic":
        st["plan"] = ctx.plan(mj.TRIANGLE, R, S, T)
    elif f not in ("adhoc", "distinct"):
        st["plan"] = ctx.plan(mj.LINEAR, R, S, T, a_domain)
    return st


def run(st):
    f = st["family"]
    if f == "batch":
        return st["batch"].run()
    ctx, R, S, T, a = st["ctx"], st["R"], st["S"], st["T"], st["a_domain"]
    if f == "adhoc":
        return ctx.linear3_count(R, S, T, a)
    if f == "distinct":
        return ctx.linear3_distinct(R, S, T, a, seed=FM_SEED)
    if f == "materialize":
        return ctx.linear3_materialize(R, S, T, first=st["first"], out=st["out"])
    p = st["plan"]
    if f == "cyclic":
        call = ctx.cascade2_count if p.algo == mj.ALGO_CASCADE else None
        return call(mj.TRIANGLE, R, S, T, plan=p) if call else ctx.triangle3_count(R, S, T, plan=p)
    if f == "cascade" or p.algo in (mj.ALGO_CASCADE, mj.ALGO_STAR_CASCADE):
        return ctx.cascade2_count(mj.LINEAR, R, S, T, a, plan=p)
    return ctx.linear3_count(R, S, T, a, plan=p)


def work(case):
    """Bytes: every relation read once, the result written once.  Operations:
    one addition per tuple (an aggregate touches every tuple at least once)."""
    f = case["family"]
    if f == "batch":
        span = case["hi"] - case["lo"]
        mean = (10 ** case["hi"] - 10 ** case["lo"]) / (span * math.log(10)) if span else 10 ** case["hi"]
        tuples = case["count"] * mean * 1.5      # half of the relations are symmetrised
        return dict(bytes=8 * tuples + case["count"] / 2 * mean / 2, flops=3 * tuples)
    if f == "cyclic" and case["shape"] != "three":
        return dict(bytes=16 * case["edges"] + 8, flops=6 * case["edges"])
    sizes = [case["n_r"], case["n_s"], case["n_t"]]
    read = 8 * (sizes[0] if case.get("same") and f != "hashed" else sum(sizes[:2]) + sizes[2] / 2)
    out = {"cyclic": 8, "distinct": 72 * case.get("domain", 0),
           "materialize": 16 * case.get("rows", 0)}.get(f, 8 * case.get("a_domain", case.get("domain", 0)))
    return dict(bytes=read + out, flops=sum(sizes))


# ------------------------------------------------------- exact results (torch)
def _ids(*cols):
    """The columns' values numbered together from 0."""
    u, inv = torch.unique(torch.cat(cols), return_inverse=True)
    return u.numel(), torch.split(inv, [c.numel() for c in cols])


def _exact_counts(R, S, T, a_domain):
    nb, (rb, sb) = _ids(R[:, 1], S[:, 0])
    nc, (sc, tc) = _ids(S[:, 1], T[:, 0])
    deg = torch.bincount(tc, minlength=nc)
    w = torch.zeros(nb, dtype=torch.int64, device=DEV).index_add_(0, sb, deg[sc])
    return torch.zeros(a_domain, dtype=torch.int64, device=DEV).index_add_(0, R[:, 0].long(), w[rb])


def _expand(starts, lens, lo, hi):
    """For the concatenation of ranges [starts, starts + lens): items [lo, hi) as (range, element)."""
    off = torch.cumsum(lens, 0)
    p = torch.arange(lo, hi, device=DEV)
    i = torch.searchsorted(off, p, right=True)
    return i, starts[i] + (p - (off[i] - lens[i]))


def _exact_cyclic(R, S, T, most=3 << 30):
    nb, (rb, sb) = _ids(R[:, 1], S[:, 0])
    start = torch.cumsum(torch.bincount(rb, minlength=nb), 0)
    lens = torch.bincount(rb, minlength=nb)[sb]
    total = int(lens.sum())
    if total > most:
        return None
    ra = R[:, 0][torch.argsort(rb)].long()
    first = start[sb] - lens
    tk = torch.sort((T[:, 0].long() << 32) | (T[:, 1].long() & M32)).values
    found = 0
    for lo in range(0, total, 1 << 26):
        i, e = _expand(first, lens, lo, min(total, lo + (1 << 26)))
        key = (S[:, 1][i].long() << 32) | (ra[e] & M32)
        found += int((torch.searchsorted(tk, key, right=True) - torch.searchsorted(tk, key)).sum())
    return torch.tensor([found], dtype=torch.int64, device=DEV)


def _exact_triangles(E, most=3 << 30):
    """A symmetric simple relation: edges kept towards the higher (degree, id), wedges closed."""
    x, y = E[:, 0].long(), E[:, 1].long()
    deg = torch.bincount(x)
    up = (deg[x] < deg[y]) | ((deg[x] == deg[y]) & (x < y))
    key = torch.sort((x[up] << 32) | y[up]).values
    x, y = key >> 32, key & M32
    out = torch.bincount(x, minlength=deg.numel())
    lens, first = out[x], (torch.cumsum(out, 0) - out)[x]
    total = int(lens.sum())
    if total > most:
        return None
    found = 0
    for lo in range(0, total, 1 << 26):
        i, e = _expand(first, lens, lo, min(total, lo + (1 << 26)))
        k = (y[i] << 32) | y[e]
        at = torch.searchsorted(key, k).clamp(max=key.numel() - 1)
        found += int((key[at] == k).sum())
    return torch.tensor([6 * found], dtype=torch.int64, device=DEV)


def _exact_rows(R, S, T, first, rows):
    """Result tuples at positions [first, first + rows) in nested-loop order, and the total."""
    nb, (rb, sb) = _ids(R[:, 1], S[:, 0])
    nc, (sc, tc) = _ids(S[:, 1], T[:, 0])
    so, to = torch.argsort(sb, stable=True), torch.argsort(tc, stable=True)
    ns, nt = torch.bincount(sb, minlength=nb), torch.bincount(tc, minlength=nc)
    per_s = nt[sc][so]
    ps = torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), torch.cumsum(per_s, 0)])
    s0 = torch.cumsum(ns, 0) - ns
    per_r = (ps[s0 + ns] - ps[s0])[rb]
    total = int(per_r.sum())
    out = torch.zeros((rows, 4), dtype=torch.int32, device=DEV)
    t0 = torch.cumsum(nt, 0) - nt
    for lo in range(first, min(total, first + rows), 1 << 24):
        hi = min(total, first + rows, lo + (1 << 24))
        j, k = _expand(ps[s0[rb]], per_r, lo, hi)        # k: position in S's concatenated matches
        i = torch.searchsorted(ps, k, right=True) - 1
        s = so[i]
        t = to[t0[sc[s]] + (k - ps[i])]
        out[lo - first:hi - first] = torch.stack([R[j, 0], R[j, 1], S[s, 1], T[t, 1]], dim=1)
    return out, torch.tensor([total], dtype=torch.int64, device=DEV)


def _mix(x, seed):
    """MurmurHash3's 32-bit finaliser of x xor seed."""
    h = (x.long() & M32) ^ seed
    h = ((h ^ (h >> 16)) * 0x85EBCA6B) & M32
    h = ((h ^ (h >> 13)) * 0xC2B2AE35) & M32
    return h ^ (h >> 16)


def _or_by(key, words, groups):
    """OR of the rows of `words` per key."""
    order = torch.argsort(key)
    key, words = key[order], words[order]
    step = 1
    most = int(torch.bincount(key).max())
    while step < most:                           # every row ORs the 2^k rows from its own on
        same = key[step:] == key[:-step]
        words[:-step] |= words[step:].clone() * same[:, None]
        step *= 2
    out = torch.zeros((groups, 16), dtype=torch.int32, device=DEV)
    head = torch.ones_like(key, dtype=torch.bool)
    head[1:] = key[1:] != key[:-1]
    out[key[head]] = words[head]
    return out


def _exact_distinct(R, S, T, a_domain):
    nb, (rb, sb) = _ids(R[:, 1], S[:, 0])
    nc, (sc, tc) = _ids(S[:, 1], T[:, 0])
    h = _mix(T[:, 1], FM_SEED)
    rest = h >> 4
    low = rest & -rest
    bit = torch.where(rest == 0, torch.full_like(low, 1 << 28), low)
    words = torch.zeros((tc.numel(), 16), dtype=torch.int32, device=DEV)
    words[torch.arange(tc.numel(), device=DEV), h & 15] = bit.to(torch.int32)
    sk = _or_by(tc, words, nc)
    sk = _or_by(sb, sk[sc], nb)
    sk = _or_by(R[:, 0].long(), sk[rb], a_domain)
    w = sk.long() & M32
    zeros = torch.zeros_like(w)
    run = torch.ones_like(w, dtype=torch.bool)
    for b in range(32):
        run &= ((w >> b) & 1) == 1
        zeros += run
    est = 16.0 / 0.77351 * torch.pow(2.0, zeros.sum(1).double() / 16.0)
    return sk, torch.where((w != 0).any(1), est, torch.zeros_like(est))


def exact(case, seed):
    f = case["family"]
    if f == "batch":
        outs = []
        for kind, R, S, T, a in _batch_relations(case, seed):
            outs.append(_exact_counts(R, S, T, a) if kind == mj.LINEAR else _exact_triangles(R))
        return outs
    R, S, T, a = _relations(case, seed)
    if f == "cyclic":
        return _exact_cyclic(R, S, T) if case["shape"] == "three" else _exact_triangles(R)
    if f == "distinct":
        return _exact_distinct(R, S, T, a)
    if f == "materialize":
        return _exact_rows(R, S, T, case["first"], case["rows"])
    return _exact_counts(R, S, T, a)
