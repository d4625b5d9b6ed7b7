// Cyclic three-way join R(A,B) |x| S(B,C) |x| T(C,A), total count (Sec. 5).
//
// Every relation is turned into 64-bit keys of mixed 32-bit values and
// sorted (radix.hip):  R -> (m(b), m(a)),  T -> (m(c), m(a)),  S -> (m(b), m(c))
// and a second copy S' -> (m(c), m(b)).  m is a bijection of the 32-bit keys,
// so equal mixed values mean equal keys and every join predicate can be
// evaluated on mixed values.  After sorting, R's tuples with one B value form
// a contiguous list ordered by m(a), and so do T's tuples with one C value.
//
// The paper keeps a partition R' of R on chip and streams S' and T' past it
// (Sec. 5.1).  Here the unit kept on chip is one relation's list for one
// join value, and every S tuple is handled once, by its shorter list:
//   * pass 1 stages R's list of b and, for the s(b, c) whose T list is
//     strictly shorter, streams T's list of c past it;
//   * pass 2 stages T's list of c and, for the remaining s (R's list not
//     longer), streams R's list of b past it.
// In each pass:
//   * k_tri_light : one wave per group whose staged list has at most
//                   TRI_LIGHT_X tuples (its LDS table maps m(a) to a
//                   multiplicity);
//   * k_tri_heavy : staged lists of hub values are cut into slices of at
//                   most TRI_HEAVY_X tuples by ranges of m(a) -- the share on
//                   A -- and the groups into ranges; one workgroup per
//                   (slice, range) streams the part of each iterated list that
//                   falls in the slice's A range.
// Work items come from device queues filled by k_tri_classify.  Each wave
// sums its counts in registers and adds them to the total once.
#include "mj_kernels.h"

namespace mj {

// ------------------------------------------------------- runs of equal keys
__device__ __forceinline__ int run_find_job(const RunLaunch& L, uint32_t tile) {
    int j = 0;
#pragma unroll
    for (int q = 1; q < RUN_MAX_JOBS; ++q)
        if (q < L.njobs && tile >= L.job[q].tile_begin) j = q;
    return j;
}

// The tile's keys, wave w holding its w-th part, 64 keys a round, and the
// ballots of the run heads.  Returns the wave's number of heads.
constexpr int RUN_ROUNDS = RUN_TILE / RUN_THREADS;
__device__ __forceinline__ uint32_t run_heads(const RunJob& J, uint64_t beg, unsigned long long (&key)[RUN_ROUNDS],
                                              unsigned long long (&heads)[RUN_ROUNDS]) {
    const uint32_t lane = lane_id();
    const uint64_t at = beg + threadIdx.x / WAVE * (RUN_ROUNDS * WAVE) + lane;
    unsigned long long prev[RUN_ROUNDS];
#pragma unroll
    for (int k = 0; k < RUN_ROUNDS; ++k) {
        const uint64_t i = at + k * WAVE;
        key[k] = i < J.n ? J.keys[i] : 0ull;
        prev[k] = lane == 0 && i > 0 && i < J.n ? J.keys[i - 1] : 0ull;
    }
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < RUN_ROUNDS; ++k) {
        const uint64_t i = at + k * WAVE;
        const uint32_t hi = (uint32_t)(key[k] >> 32);
        const uint32_t up = __shfl_up(hi, 1, WAVE);
        const uint32_t before = lane == 0 ? (uint32_t)(prev[k] >> 32) : up;
        heads[k] = __ballot(i < J.n && (i == 0 || hi != before));
        c += (uint32_t)__popcll(heads[k]);
    }
    return c;
}

MJ_KERNEL(k_run_count, RUN_THREADS, RunLaunch) {
    __shared__ uint32_t wsum[RUN_THREADS / WAVE];
    if (vg.bid == 0) {                               // before the launches that count into them
        for (uint32_t w = threadIdx.x; w < A.nclear; w += blockDim.x) A.clear[w] = 0;
        if (A.zero && threadIdx.x == 0) *A.zero = 0;
    }
    const RunJob& J = A.job[run_find_job(A, vg.bid)];
    const uint32_t tile = vg.bid - J.tile_begin;
    unsigned long long key[RUN_ROUNDS], heads[RUN_ROUNDS];
    const uint32_t c = run_heads(J, uint64_t(tile) * RUN_TILE, key, heads);
    if (lane_id() == 0) wsum[threadIdx.x / WAVE] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int q = 0; q < RUN_THREADS / WAVE; ++q) t += wsum[q];
        J.part[tile] = t;
    }
}

// Every tile numbers its runs from the heads before it and writes each run's
// key, start and directory entries: a round of 64 keys knows the prefix before
// it from the key before it, so the directory needs no pass of its own, and
// its lanes write the entries side by side (two arrays of 2^22 keys: 87 us for
// 4000 runs each and 50 us for 2^18; each head filling its own gap 632 and
// 80 us).  (As separate
// flag, scan, compact and directory passes the four arrays of a join of 10^6
// tuples took 26 launches and 0.25 ms; two launches and 62 us now.)
MJ_KERNEL(k_run_emit, RUN_THREADS, RunLaunch) {
    __shared__ uint32_t wsum[RUN_THREADS / WAVE], wbefore[RUN_THREADS / WAVE];
    const RunJob& J = A.job[run_find_job(A, vg.bid)];
    const uint32_t tile = vg.bid - J.tile_begin, lane = lane_id(), w = threadIdx.x / WAVE;
    const uint64_t beg = uint64_t(tile) * RUN_TILE;
    unsigned long long key[RUN_ROUNDS], heads[RUN_ROUNDS];
    const uint32_t c = run_heads(J, beg, key, heads);
    uint32_t b = 0;
    if (A.scanned) {
        b = threadIdx.x == 0 ? J.part[tile] : 0u;
    } else {
        for (uint32_t t = threadIdx.x; t < tile; t += blockDim.x) b += J.part[t];
    }
    b = wave_sum_u32(b);
    if (lane == 0) { wsum[w] = c; wbefore[w] = b; }
    __syncthreads();
    uint32_t r = 0, end = 0;                          // runs before this wave's part, and before the next tile
    for (uint32_t q = 0; q < RUN_THREADS / WAVE; ++q) {
        r += wbefore[q] + (q < w ? wsum[q] : 0u);
        end += wbefore[q] + wsum[q];
    }
    const uint64_t at = beg + w * (RUN_ROUNDS * WAVE) + lane;
    const unsigned long long lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    uint32_t d0 = 0;                                  // the first directory entry not written before this round
    if (J.dir && at - lane > 0 && at - lane < J.n) d0 = top_bits((uint32_t)(J.keys[at - lane - 1] >> 32), J.bits) + 1u;
#pragma unroll
    for (int k = 0; k < RUN_ROUNDS; ++k) {
        const uint64_t i = at + k * WAVE;
        const uint32_t hi = (uint32_t)(key[k] >> 32);
        if (J.dir && i - lane < J.n) {                // uniform over the wave
            // entries d0 up to the last key's prefix, one a lane: the first of
            // these keys with that prefix or a greater one is a head
            const uint32_t pk = i < J.n ? top_bits(hi, J.bits) : 0xFFFFFFFFu;
            const uint32_t last = wave_read(pk, (int)min<uint64_t>(J.n - (i - lane), WAVE) - 1);
            for (; d0 <= last; d0 += WAVE) {
                const uint32_t p = d0 + lane;
                int j = 0;
#pragma unroll
                for (int step = WAVE / 2; step > 0; step /= 2)
                    if ((uint32_t)__shfl((int)pk, j + step - 1, WAVE) < p) j += step;
                if (p <= last) J.dir[p] = r + (uint32_t)__popcll(heads[k] & ((1ull << j) - 1ull));
            }
            d0 = last + 1u;
        }
        if (i < J.n && J.low) J.low[i] = (uint32_t)key[k];
        if ((heads[k] >> lane) & 1ull) {
            const uint32_t run = r + (uint32_t)__popcll(heads[k] & lt_mask);
            J.run_key[run] = hi;
            J.run_start[run] = (uint32_t)i;
        }
        r += (uint32_t)__popcll(heads[k]);
    }
    if (tile != J.ntiles - 1) return;
    if (threadIdx.x == 0) {
        J.run_start[end] = (uint32_t)J.n;
        *J.nruns = end;
    }
    if (J.dir) {                                      // the prefixes after the last run's
        const uint32_t p0 = J.n == 0 ? 0u : top_bits((uint32_t)(J.keys[J.n - 1] >> 32), J.bits) + 1u;
        for (uint32_t p = p0 + threadIdx.x; p <= (1u << J.bits); p += blockDim.x) J.dir[p] = end;
    }
}

// --------------------------------------------------------------- classify
// Light: R list of b short and S group small -> one wave.  Heavy: otherwise
// -> (slice of R's list) x (range of the S group) workgroup items, counted
// per group here and enumerated through the counts before each group.
// `range` is the S tuples of an item: TRI_HEAVY_S, more only where a group
// would have over 2^TRI_HEAVY_RANGE_BITS ranges, so that the items of any
// relations of under 2^32 tuples stay within HEAVY_SHIFT bits (a hub of 2^27
// tuples on both sides has 2^32 of them).
constexpr uint32_t TRI_HEAVY_RANGE_BITS = 16;
__device__ __forceinline__ void heavy_shape(uint32_t x, uint32_t gn, uint32_t share, uint32_t& nsl, uint32_t& nsr,
                                            uint32_t& range) {
    nsl = (uint32_t)((uint64_t(x) + TRI_HEAVY_X - 1) / TRI_HEAVY_X);
    nsl = max(nsl, min(share, (uint32_t)((uint64_t(x) + 63) / 64)));
    range = TRI_HEAVY_S;
    while (gn > uint64_t(range) << TRI_HEAVY_RANGE_BITS) range *= 2;
    nsr = (uint32_t)((uint64_t(gn) + range - 1) / range);
}

// Groups are appended with one atomic per workgroup and round of 1024 groups
// (one per wave serialised on the counter's address: 370 us a pass at scale
// 22).  A light entry carries its group's run and its staged list's run.
// Heavy groups and their items are counted in one 64-bit word, so a heavy
// group learns its place and the items before it from the same atomic.
MJ_KERNEL(k_tri_classify, 256, TriClassifyPair) {
    __shared__ uint32_t wl[256 / WAVE], lbase;
    __shared__ unsigned long long wh[256 / WAVE], hbase;
    const bool second = vg.bid >= A.per;
    const TriClassifyArgs& C = A.pass[second ? 1 : 0];
    const uint32_t bid = second ? vg.bid - A.per : vg.bid;
    const uint64_t ng = *C.Grp.nruns;
    const int lane = lane_id(), w = threadIdx.x / WAVE;
    for (uint64_t g0 = bid * 1024ull; g0 < ng; g0 += A.per * 1024ull) {      // uniform over the block
        uint32_t key[4], run[4], nlight = 0;
        unsigned long long items[4], nheavy = 0;
        bool live[4], light[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint64_t g = g0 + u * 256 + threadIdx.x;
            live[u] = g < ng;
            key[u] = live[u] ? C.Grp.run_key[g] : 0u;
        }
        run_find4(C.Stg, key, live, run);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            light[u] = false;
            items[u] = 0;
            if (run[u] == 0xFFFFFFFFu) continue;
            const uint64_t g = g0 + u * 256 + threadIdx.x;
            const uint32_t x = C.Stg.run_start[run[u] + 1] - C.Stg.run_start[run[u]];
            const uint32_t gn = C.Grp.run_start[g + 1] - C.Grp.run_start[g];
            light[u] = x <= TRI_LIGHT_X && gn <= TRI_LIGHT_S;
            if (light[u]) {
                ++nlight;
            } else {
                uint32_t nsl, nsr, range;
                heavy_shape(x, gn, C.share, nsl, nsr, range);
                items[u] = (unsigned long long)nsl * nsr;
                nheavy += (1ull << HEAVY_SHIFT) | items[u];
            }
        }
        uint32_t vl = nlight;                         // inclusive prefixes over the wave
        unsigned long long vh = nheavy;
#pragma unroll
        for (int off = 1; off < WAVE; off <<= 1) {
            const uint32_t yl = __shfl_up(vl, off, WAVE);
            const unsigned long long yh = __shfl_up(vh, off, WAVE);
            if (lane >= off) { vl += yl; vh += yh; }
        }
        if (lane == WAVE - 1) { wl[w] = vl; wh[w] = vh; }
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t tl = 0;
            unsigned long long th = 0;
            for (int q = 0; q < 256 / WAVE; ++q) { tl += wl[q]; th += wh[q]; }
            lbase = tl ? atomicAdd(C.nlight, tl) : 0u;
            hbase = th ? atomicAdd(C.heavy, th) : 0ull;
        }
        __syncthreads();
        uint32_t at = lbase + vl - nlight;
        unsigned long long hat = hbase + vh - nheavy;
        for (int q = 0; q < w; ++q) { at += wl[q]; hat += wh[q]; }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t g = (uint32_t)(g0 + u * 256 + threadIdx.x);
            if (light[u]) C.light[at++] = make_uint2(g, run[u]);
            if (items[u]) {
                const uint32_t hg = (uint32_t)(hat >> HEAVY_SHIFT);
                C.heavy_group[hg] = g;
                C.heavy_off[hg] = hat & ((1ull << HEAVY_SHIFT) - 1ull);
                hat += (1ull << HEAVY_SHIFT) | items[u];
            }
        }
        __syncthreads();                              // the shared words are used again
    }
}

// ------------------------------------------------------------- staged lists
// A staged list lies in LDS as it is, sorted by m(a) (at least by its top bits
// from TriJoinArgs::low_bits up; a bucket is no finer), with a directory over
// the range of its values: the values are hashes, so equal-width buckets
// hold about the same number each.  dir[bucket] = first position | number of
// entries << 16.  A lookup reads one directory word and then the bucket's
// entries (one or two), where an open-addressing table at half load made a
// wave walk as far as the longest of its 64 probe chains.  A list with equal
// entries (bags) also has run[q] = how many entries equal to val[q] start at
// q, and a lookup steps over the bucket run by run, so that a tuple repeated
// thousands of times costs one step.  Bound by the lookups'
// instructions (about one vector instruction an entry), then by the latency
// of the streamed lists.  Oriented join of the R-MAT graph of scale 22
// (1.3e10 streamed entries): light kernel 48.1 -> 8.2 ms, heavy kernel
// 24.2 -> 12.5 ms against hash tables and one list in flight.
struct ListTab {
    uint32_t* dir;
    uint32_t* val;
    uint16_t* run;
    uint32_t base, top, shift;        // bucket of a: (a - base) >> shift, when a - base <= top
    bool dup;                         // some entries are equal: `run` is set
};

// entry q into the directory; true when it equals the entry before it
__device__ __forceinline__ bool listtab_index(const ListTab& T, uint32_t q) {
    const uint32_t v = T.val[q], b = (v - T.base) >> T.shift;
    const uint32_t u = q ? T.val[q - 1] : 0u;
    const bool head = q == 0 || ((u - T.base) >> T.shift) != b;
    atomicAdd(&T.dir[b], 0x10000u + (head ? q : 0u));
    return q && u == v;
}

// run[q] of a run's first entry: the end of its run, by a binary search in
// the rest of its bucket (step by step where the bucket is not in order:
// then a value may have several runs, each counted)
__device__ __forceinline__ void listtab_run(const ListTab& T, uint32_t q, bool in_order) {
    const uint32_t v = T.val[q];
    if (q && T.val[q - 1] == v) return;
    const uint32_t d = T.dir[(v - T.base) >> T.shift];
    uint32_t lo = q + 1, hi = (d & 0xFFFFu) + (d >> 16);
    if (!in_order) {
        while (lo < hi && T.val[lo] == v) ++lo;
        hi = lo;
    }
    while (lo < hi) {
        const uint32_t m = (lo + hi) >> 1;
        if (T.val[m] == v) lo = m + 1; else hi = m;
    }
    T.run[q] = (uint16_t)(lo - q);
}

// entries equal to the four keys; every read of a step is in flight together
template <bool DUP>
__device__ __forceinline__ uint32_t listtab_count4(const ListTab& T, const uint32_t (&key)[4], const bool (&live)[4]) {
    uint32_t p[4], n[4], acc = 0, most = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t o = key[u] - T.base;
        const bool in = live[u] && o <= T.top;
        const uint32_t d = T.dir[in ? o >> T.shift : 0u];
        p[u] = d & 0xFFFFu;
        n[u] = in ? d >> 16 : 0u;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) most = max(most, n[u]);
    if constexpr (DUP) {
        uint32_t e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) e[u] = p[u] + n[u];
        bool more = most > 0;
        while (more) {
            more = false;
            uint32_t v[4], r[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) { v[u] = T.val[p[u] < e[u] ? p[u] : 0u]; r[u] = T.run[p[u] < e[u] ? p[u] : 0u]; }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (p[u] >= e[u]) continue;
                acc += v[u] == key[u] ? r[u] : 0u;
                p[u] += r[u];
                more = more || p[u] < e[u];
            }
        }
        return acc;
    }
    for (uint32_t i = 0; i < most; ++i) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = T.val[i < n[u] ? p[u] + i : 0u];
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += i < n[u] && v[u] == key[u] ? 1u : 0u;
    }
    return acc;
}

// ------------------------------------------------------- streaming lists
// One chunk of up to 64 S tuples of a group, lane j holding tuple si (when
// `valid`): each tuple's iterated list streams past the staged one.  When the
// staged list is a slice, only the part of a list in the slice's range of A
// is read: every lane finds its own list's part by two binary searches, 64
// lists at a time.  Lists of at most TRI_SHORT_LIST entries are then walked
// by their own lane; longer ones by the whole wave in pieces of 64
// consecutive entries, four pieces (of one list or of several) per step, the
// next step's pieces loaded before the present ones are looked up.  Returns
// the lane's partial sum.
template <bool DUP>
__device__ __forceinline__ unsigned long long stream_chunk(const TriJoinArgs& A, uint32_t si, bool valid,
                                                           uint32_t x, const ListTab& T, bool sliced) {
    const int lane = lane_id();
    unsigned long long acc = 0;
    uint32_t ts = 0, y = 0;
    if (!(valid && run_lookup(A.Itr, A.Grpl[si], ts, y)) ||
        (A.strict ? y >= x : y > x))                  // the other pass owns this s
        y = 0;
    if (sliced && y > 4) {                            // the part inside [base, base + top]
        uint32_t l = ts, h = ts + y, l2 = ts, h2 = ts + y;
        const uint32_t last = T.base + T.top;
        while (l < h || l2 < h2) {
            const uint32_t m = (l + h) >> 1, m2 = (l2 + h2) >> 1;
            const uint32_t k = l < h ? A.Itrl[m] : 0u, k2 = l2 < h2 ? A.Itrl[m2] : 0u;
            if (l < h) { if (k < T.base) l = m + 1; else h = m; }
            if (l2 < h2) { if (k2 <= last) l2 = m2 + 1; else h2 = m2; }
        }
        ts = l;
        y = l2 - l;
    }
    if (y > 0 && y <= TRI_SHORT_LIST) {
        const uint32_t te = ts + y;
        uint32_t key[4];
        bool live[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            live[u] = ts + u < te;
            key[u] = live[u] ? A.Itrl[ts + u] : 0u;
        }
        for (uint32_t t0 = ts; t0 < te; t0 += 4) {
            uint32_t nkey[4];
            bool nlive[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                nlive[u] = t0 + 4 + u < te;
                nkey[u] = nlive[u] ? A.Itrl[t0 + 4 + u] : 0u;
            }
            acc += listtab_count4<DUP>(T, key, live);
#pragma unroll
            for (int u = 0; u < 4; ++u) { key[u] = nkey[u]; live[u] = nlive[u]; }
        }
    }
    unsigned long long longm = __ballot(y > TRI_SHORT_LIST);
    uint32_t t = 0, te = 0;                           // the list being cut into pieces (wave-uniform)
    uint32_t key[4];
    bool live[4];
    auto fetch = [&](uint32_t (&k)[4], bool (&lv)[4]) -> bool {
        bool any = false;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (t >= te && longm) {
                const int j = __ffsll((long long)longm) - 1;
                longm &= longm - 1;
                t = wave_read(ts, j);
                te = t + wave_read(y, j);
            }
            lv[u] = t + lane < te;
            k[u] = lv[u] ? A.Itrl[t + lane] : 0u;
            any = any || t < te;
            t = min(t + WAVE, te);
        }
        return any;                                   // wave-uniform
    };
    bool more = fetch(key, live);
    while (more) {
        uint32_t nkey[4];
        bool nlive[4];
        more = fetch(nkey, nlive);
        acc += listtab_count4<DUP>(T, key, live);
#pragma unroll
        for (int u = 0; u < 4; ++u) { key[u] = nkey[u]; live[u] = nlive[u]; }
    }
    return acc;
}

// ------------------------------------------------------------- light groups
// One wave, one S group: the staged list (at most TRI_LIGHT_X entries) and its
// directory in 6.6 KB of LDS per wave, so six workgroups (24 waves) fit a CU;
// then every s(b,c) of the group streams its iterated list past it, 64 tuples
// at a time (stream_chunk).  Returns the lane's sum.
__device__ unsigned long long tri_light_group(const TriJoinArgs& A, uint2 item, ListTab T) {
    const int lane = lane_id();
    const uint32_t gs = A.Grp.run_start[item.x], ge = A.Grp.run_start[item.x + 1];
    const uint32_t rs = A.Stg.run_start[item.y], x = A.Stg.run_start[item.y + 1] - rs;
    for (uint32_t q = lane; q < x; q += WAVE) T.val[q] = A.Stgl[rs + q];
    wave_fence();
    bool dup = false;
    for (uint32_t q = lane; q < x; q += WAVE) dup = listtab_index(T, q) || dup;
    wave_fence();
    T.dup = __ballot(dup) != 0;
    unsigned long long acc = 0;
    if (T.dup) {
        for (uint32_t q = lane; q < x; q += WAVE) listtab_run(T, q, A.low_bits == 0);
        wave_fence();
        for (uint32_t c0 = gs; c0 < ge; c0 += WAVE)
            acc += stream_chunk<true>(A, c0 + lane, c0 + lane < ge, x, T, false);
    } else {
        for (uint32_t c0 = gs; c0 < ge; c0 += WAVE)
            acc += stream_chunk<false>(A, c0 + lane, c0 + lane < ge, x, T, false);
    }
    wave_fence();
    for (uint32_t q = lane; q < x; q += WAVE) T.dir[T.val[q] >> T.shift] = 0;
    wave_fence();
    return acc;
}

#define TRI_LIGHT_SETUP                                                              \
    constexpr int NW = TRI_THREADS / WAVE;                                           \
    __shared__ uint32_t tdir[NW][1u << TRI_LIGHT_DIR_BITS];                          \
    __shared__ uint32_t tval[NW][TRI_LIGHT_X];                                       \
    __shared__ uint16_t trun[NW][TRI_LIGHT_X];                                       \
    const int w = threadIdx.x / WAVE, lane = lane_id();                              \
    const ListTab T{tdir[w], tval[w], trun[w], 0u, 0xFFFFFFFFu, 32 - TRI_LIGHT_DIR_BITS, false}; \
    for (uint32_t s = lane; s < (1u << TRI_LIGHT_DIR_BITS); s += WAVE) T.dir[s] = 0; \
    wave_fence();

// Light items are taken a run at a time from TRI_QUEUES queues, each over its
// own part of the items with its counter on a cache line of its own: atomics
// on one address are served one after another (about 12 ns each), and one
// counter for all waves took 0.3 ms a pass for the 65,536 groups of a join of
// 10^6 tuples.  A run is a quarter of a wave's fair share, at least
// TRI_LIGHT_GRAB_MIN and at most TRI_LIGHT_GRAB items.  A workgroup starts at
// queue (its number modulo TRI_QUEUES); when that one is empty each lane looks
// at one counter, and the wave goes on with the next queue that has items.
constexpr uint32_t TRI_LIGHT_GRAB = 16, TRI_LIGHT_GRAB_MIN = 4;
static_assert(TRI_QUEUES <= WAVE, "one lane looks at one queue");

__device__ __forceinline__ uint32_t light_grab(unsigned long long nitems, unsigned long long waves) {
    const unsigned long long g = nitems / (4ull * waves);
    return (uint32_t)(g < TRI_LIGHT_GRAB_MIN ? TRI_LIGHT_GRAB_MIN : (g > TRI_LIGHT_GRAB ? TRI_LIGHT_GRAB : g));
}

// The next run [it, end) of items for the wave, or false when every queue is
// empty.  `q` is the wave's present queue; `counters` hold the items already
// taken of each queue (they may run past its length).  Wave-uniform.
__device__ __forceinline__ bool light_next_run(uint32_t* counters, unsigned long long nitems, uint32_t grab,
                                               uint32_t& q, unsigned long long& it, unsigned long long& end) {
    const uint32_t lane = lane_id();
    while (true) {
        const unsigned long long q0 = nitems * q / TRI_QUEUES, q1 = nitems * (q + 1) / TRI_QUEUES;
        uint32_t t = 0;
        if (lane == 0) t = atomicAdd(&counters[q * TRI_QUEUE_PAD], grab);
        t = __shfl(t, 0, WAVE);
        if (q0 + t < q1) {
            it = q0 + t;
            end = min(it + grab, q1);
            return true;
        }
        // lane l looks at queue q + l (a stale value only costs one more try)
        const uint32_t o = (q + lane) % TRI_QUEUES;
        const unsigned long long len = nitems * (o + 1) / TRI_QUEUES - nitems * o / TRI_QUEUES;
        const uint32_t taken = lane == 0 ? 0xFFFFFFFFu : *(volatile uint32_t*)&counters[o * TRI_QUEUE_PAD];
        const unsigned long long has = __ballot(lane < TRI_QUEUES && lane > 0 && taken < len);
        if (has == 0) return false;
        q = (q + (uint32_t)__ffsll((long long)has) - 1u) % TRI_QUEUES;
    }
}

// Both passes in one launch: a wave that finds pass 0's queues empty goes on
// with pass 1's.
MJ_KERNEL(k_tri_light, TRI_THREADS, TriJoinPair) {
    TRI_LIGHT_SETUP
    (void)lane;
    unsigned long long acc = 0;
    for (int pass = 0; pass < 2; ++pass) {
        const TriJoinArgs& P = A.pass[pass];
        const uint32_t nitems = *P.nlight;
        const uint32_t grab = light_grab(nitems, (unsigned long long)vg.nblk * (TRI_THREADS / WAVE));
        unsigned long long it = 0, end = 0;
        uint32_t q = vg.bid % TRI_QUEUES;
        while (true) {
            if (it >= end && !light_next_run(P.light_next, nitems, grab, q, it, end)) break;   // wave-uniform
            acc += tri_light_group(P, P.light[it], T);
            ++it;
        }
    }
    block_add_u64(A.pass[0].total, acc);
}

// ------------------------------------------------------------- heavy groups
// One workgroup, one item: a slice of a hub's staged list (at most TRI_HEAVY_X
// entries) and its directory in 28 KB of LDS, then the item's S tuples stream
// their iterated lists past it (only the part in the slice's range of A when
// the staged list is sliced).  Waves take chunks of S tuples from a workgroup
// counter.  Eight waves and 2048 entries: with 16 waves and 4096 entries the
// many lists of 449 to 1,100 entries left waves idle (17.3 -> 12.5 ms at scale
// 22, oriented).
struct BlockTable {
    uint32_t* dir;
    uint32_t* val;
    uint16_t* run;
    uint32_t* dup;
    uint32_t* chunk;                  // next chunk of the item's S tuples
};

// last h in [0, n) with off[h] <= it, given off[0] <= it: 64 entries a round
__device__ __forceinline__ uint32_t wave_last_le(const unsigned long long* off, uint32_t n, unsigned long long it) {
    const uint32_t lane = lane_id();
    uint32_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const uint32_t step = (hi - lo + WAVE - 1) / WAVE;
        const uint32_t k = lo + lane * step;
        const unsigned long long bal = __ballot(k < hi && off[k] <= it);
        lo += (uint32_t)(63 - __clzll((long long)bal)) * step;
        hi = min(hi, lo + step);
    }
    return lo;
}

__device__ unsigned long long tri_heavy_item(const TriJoinArgs& A, unsigned long long it, const BlockTable& B) {
    const int lane = lane_id();
    // item -> (heavy group, slice of the staged list, range of the group)
    const uint32_t lo = wave_last_le(A.heavy_off, (uint32_t)(*A.heavy >> HEAVY_SHIFT), it);
    const uint32_t g = A.heavy_group[lo];
    const unsigned long long local = it - A.heavy_off[lo];
    uint32_t rs = 0, x = 0;
    run_lookup(A.Stg, A.Grp.run_key[g], rs, x);
    const uint32_t gs = A.Grp.run_start[g], gn = A.Grp.run_start[g + 1] - gs;
    uint32_t nsl, nsr, range;
    heavy_shape(x, gn, A.share, nsl, nsr, range);
    const uint32_t sa = (uint32_t)(local / nsr), sb = (uint32_t)(local % nsr);
    const uint32_t r0 = rs + (uint32_t)((uint64_t)x * sa / nsl);
    const uint32_t r1 = rs + (uint32_t)((uint64_t)x * (sa + 1) / nsl);
    const uint32_t s0 = gs + sb * range, s1 = gs + (uint32_t)min<uint64_t>(gn, (uint64_t(sb) + 1) * range);
    if (r0 == r1) return 0;                           // uniform across the block
    const uint32_t len = r1 - r0;
    const uint32_t low = (1u << A.low_bits) - 1u;      // the bits the lists are not ordered by
    ListTab T{B.dir, B.val, B.run, A.Stgl[r0] & ~low, 0u, 0u, false};
    T.top = (A.Stgl[r1 - 1] | low) - T.base;
    const uint32_t width = 32u - (uint32_t)__clz((int)(T.top | 1u));           // bits of the largest offset
    T.shift = max(A.low_bits, width > TRI_HEAVY_DIR_BITS ? width - TRI_HEAVY_DIR_BITS : 0u);
    for (uint32_t q = threadIdx.x; q < len; q += blockDim.x) T.val[q] = A.Stgl[r0 + q];
    for (uint32_t q = threadIdx.x; q < (1u << TRI_HEAVY_DIR_BITS); q += blockDim.x) T.dir[q] = 0;
    __syncthreads();
    bool dup = false;
    for (uint32_t q = threadIdx.x; q < len; q += blockDim.x) dup = listtab_index(T, q) || dup;
    if (dup) *B.dup = 1;
    __syncthreads();
    T.dup = *B.dup != 0;                              // uniform across the block
    if (T.dup) {
        for (uint32_t q = threadIdx.x; q < len; q += blockDim.x) listtab_run(T, q, A.low_bits == 0);
        __syncthreads();
    }
    const bool sliced = nsl > 1;
    // chunks of at most 64 S tuples, smaller ones while a wave would get fewer than two
    const uint32_t per = min((uint32_t)WAVE, max(8u, (s1 - s0) / (2 * (blockDim.x / WAVE))));
    unsigned long long acc = 0;
    while (true) {
        uint32_t c = 0;
        if (lane == 0) c = atomicAdd(B.chunk, 1u);
        const uint32_t c0 = s0 + __shfl(c, 0, WAVE) * per;
        if (c0 >= s1) break;                          // wave-uniform
        const uint32_t si = c0 + lane;
        const bool valid = (uint32_t)lane < per && si < s1;
        acc += T.dup ? stream_chunk<true>(A, si, valid, x, T, sliced) : stream_chunk<false>(A, si, valid, x, T, sliced);
    }
    return acc;
}

#define TRI_HEAVY_SETUP                                                   \
    __shared__ uint32_t hdir[1u << TRI_HEAVY_DIR_BITS];                   \
    __shared__ uint32_t hval[TRI_HEAVY_X];                                \
    __shared__ uint16_t hrun[TRI_HEAVY_X];                                \
    __shared__ uint32_t hdup, hchunk;                                     \
    const BlockTable B{hdir, hval, hrun, &hdup, &hchunk};

MJ_KERNEL(k_tri_heavy, TRI_HEAVY_THREADS, TriJoinPair) {
    (void)vg;
    TRI_HEAVY_SETUP
    __shared__ unsigned long long s_item;
    unsigned long long acc = 0;
    for (int pass = 0; pass < 2; ++pass) {
        const TriJoinArgs& P = A.pass[pass];
        const unsigned long long nitems = *P.heavy & ((1ull << HEAVY_SHIFT) - 1ull);
        while (nitems) {                              // uniform across the block
            __syncthreads();
            if (threadIdx.x == 0) { s_item = atomicAdd(P.heavy_next, 1ull); hchunk = 0; hdup = 0; }
            __syncthreads();
            const unsigned long long it = s_item;
            if (it >= nitems) break;
            acc += tri_heavy_item(P, it, B);
        }
    }
    block_add_u64(A.pass[0].total, acc);
}

// ------------------------------------------------------------- batches
// Every cyclic join of a batch prepared its own queues; one persistent
// launch serves all of them.  Global item k -> (join j, local item) through
// the exclusive prefix of the per-join item counts.
__device__ __forceinline__ uint32_t batch_join_of(const unsigned long long* base, uint32_t njoins,
                                                  unsigned long long k) {
    uint32_t lo = 0, hi = njoins;                     // last j with base[j] <= k
    while (hi - lo > 1) { uint32_t m = (lo + hi) >> 1; if (base[m] <= k) lo = m; else hi = m; }
    return lo;
}

__global__ void __launch_bounds__(TRI_THREADS)
k_tri_light_batch(TriBatchArgs Bt) {
    TRI_LIGHT_SETUP
    const unsigned long long nitems = Bt.light_base[Bt.njoins];
    const uint32_t grab = light_grab(nitems, (unsigned long long)gridDim.x * (TRI_THREADS / WAVE));
    unsigned long long it = 0, end = 0, acc = 0;
    uint32_t cur = 0;                                 // the join whose count acc holds
    uint32_t q = blockIdx.x % TRI_QUEUES;
    while (true) {
        if (it >= end && !light_next_run(Bt.light_next, nitems, grab, q, it, end)) break;   // wave-uniform
        const uint32_t j = batch_join_of(Bt.light_base, Bt.njoins, it);
        if (j != cur) {                               // a run may span joins: add the last one's count
            acc = wave_sum_u64(acc);
            if (lane == 0 && acc) atomicAdd(Bt.joins[cur].total, acc);
            acc = 0;
            cur = j;
        }
        const TriJoinArgs& A = Bt.joins[j];
        acc += tri_light_group(A, A.light[it - Bt.light_base[j]], T);
        ++it;
    }
    acc = wave_sum_u64(acc);
    if (lane == 0 && acc) atomicAdd(Bt.joins[cur].total, acc);
}

__global__ void __launch_bounds__(TRI_HEAVY_THREADS)
k_tri_heavy_batch(TriBatchArgs Bt) {
    TRI_HEAVY_SETUP
    __shared__ unsigned long long s_bitem;
    __shared__ unsigned long long s_sum;
    const unsigned long long nitems = Bt.heavy_base[Bt.njoins];
    while (true) {
        __syncthreads();
        if (threadIdx.x == 0) { s_bitem = atomicAdd(Bt.heavy_next, 1ull); hchunk = 0; hdup = 0; s_sum = 0; }
        __syncthreads();
        const unsigned long long it = s_bitem;
        if (it >= nitems) break;
        const uint32_t j = batch_join_of(Bt.heavy_base, Bt.njoins, it);
        const TriJoinArgs& A = Bt.joins[j];
        unsigned long long acc = tri_heavy_item(A, it - Bt.heavy_base[j], B);
        acc = wave_sum_u64(acc);
        if (lane_id() == 0 && acc) atomicAdd(&s_sum, acc);
        __syncthreads();
        if (threadIdx.x == 0 && s_sum) atomicAdd(A.total, s_sum);
    }
}

// per-join item counts of a batch -> exclusive prefixes, and the batch's
// queue counters cleared (one wave, a join per lane and round)
__global__ void __launch_bounds__(WAVE) k_tri_batch_prefix(TriBatchArgs Bt) {
    const uint32_t lane = threadIdx.x;
    for (uint32_t i = lane; i < TRI_QUEUES * TRI_QUEUE_PAD; i += WAVE) Bt.light_next[i] = 0;
    if (lane == 0) *Bt.heavy_next = 0;
    unsigned long long l0 = 0, h0 = 0;
    for (uint32_t j0 = 0; j0 < Bt.njoins; j0 += WAVE) {
        const uint32_t j = j0 + lane;
        const unsigned long long nl = j < Bt.njoins ? *Bt.joins[j].nlight : 0ull;
        const unsigned long long nh = j < Bt.njoins ? *Bt.joins[j].heavy & ((1ull << HEAVY_SHIFT) - 1ull) : 0ull;
        unsigned long long l = nl, h = nh;
#pragma unroll
        for (int off = 1; off < WAVE; off <<= 1) {
            const unsigned long long yl = __shfl_up(l, off, WAVE), yh = __shfl_up(h, off, WAVE);
            if ((int)lane >= off) { l += yl; h += yh; }
        }
        if (j < Bt.njoins) { Bt.light_base[j] = l0 + l - nl; Bt.heavy_base[j] = h0 + h - nh; }
        l0 += __shfl(l, WAVE - 1, WAVE);
        h0 += __shfl(h, WAVE - 1, WAVE);
    }
    if (lane == 0) { Bt.light_base[Bt.njoins] = l0; Bt.heavy_base[Bt.njoins] = h0; }
}

// ----------------------------------------------- cascade, cyclic second join
// For every (a, c) of I = R |x| S: the multiplicity of (c, a) in T, found in
// T's sorted list of m(c) by binary search on m(a).
// A pair's lookup is a chain of dependent random reads (directory, run, its
// start, the searches for the first and last equal entry): four pairs a
// thread walk theirs together, both searches of a pair at once (the
// cascades in a batch of 64 joins: 467 -> 392 us).
MJ_KERNEL(k_cas_probe_tri, 256, CasProbeTriArgs) {
    unsigned long long acc = 0;
    const uint64_t step = 4 * uint64_t(blockDim.x);
    for (uint64_t q = vg.bid * step + threadIdx.x; q < A.n; q += vg.nblk * step) {
        uint32_t key[4], a[4], r[4], l[4], h[4], l2[4], h2[4];
        bool live[4];
        uint2 iv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) iv[u] = A.I[min<uint64_t>(q + uint64_t(u) * blockDim.x, A.n - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            live[u] = q + uint64_t(u) * blockDim.x < A.n;
            key[u] = mix32(iv[u].y, A.seed);
            a[u] = mix32(iv[u].x, A.seed);
        }
        run_find4(A.T, key, live, r);
#pragma unroll
        for (int u = 0; u < 4; ++u) {                     // run 0 stands in for a missing one
            const bool found = r[u] != 0xFFFFFFFFu;
            const uint32_t i = found ? r[u] : 0u;
            l[u] = l2[u] = A.T.run_start[i];
            const uint32_t e = A.T.run_start[i + 1];
            h[u] = h2[u] = found ? e : l[u];
        }
        bool any = true;
        while (any) {
            uint32_t k[4], k2[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (l[u] < h[u]) k[u] = (uint32_t)A.Tk[(l[u] + h[u]) >> 1];
                if (l2[u] < h2[u]) k2[u] = (uint32_t)A.Tk[(l2[u] + h2[u]) >> 1];
            }
            any = false;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t m = (l[u] + h[u]) >> 1, m2 = (l2[u] + h2[u]) >> 1;
                if (l[u] < h[u]) { if (k[u] < a[u]) l[u] = m + 1; else h[u] = m; }
                if (l2[u] < h2[u]) { if (k2[u] <= a[u]) l2[u] = m2 + 1; else h2[u] = m2; }
                any = any || l[u] < h[u] || l2[u] < h2[u];
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += l2[u] - l[u];
    }
    block_add_u64(A.total, acc);
}

}  // namespace mj
