// Star three-way join (Sec. 6, "linear star 3-way join"): the linear query
// R(A,B) |x| S(B,C) |x| T(C,D) counted per A when R and T are small
// dimension relations and S is a large fact relation.  The paper loads R and
// T on chip and streams S once past them; no partitioning of S is needed.
//
// On MI355X streaming S is a group-by on B weighted by mult_T(C):
//   W[b] = sum over s(b, c) in S of mult_T(c),   count[a] = sum over r(a, b) of W[b].
// Dimensions of at most STAR_SMALL tuples (k_star_stream, k_star_finish) are
// read by every workgroup, which builds both tables in its LDS, streams its
// contiguous chunk of S past them and adds the weights at the first R tuple
// with the same B.
//
// For larger ones the dimension tables are one-bucket multiplicity tables
// (built by the partitioner and k_dbuild of the linear path).
// R's distinct B values are numbered 0..k-1 (a prefix sum over the occupied
// slots of R's table).  "On chip" is each workgroup's LDS: one workgroup
// per CU copies T's table and R's (key, number) table there, streams its
// contiguous chunk of S, adds the weights per number in LDS and writes its
// sums once; k_star_reduce adds them up.  A random read of an L2-resident
// table costs about as much as a whole streamed tuple at these rates, which
// is why both tables are copied.  Tables larger than the LDS copies are
// probed in L2 and the sums go to global memory (exact at any size; the
// planner only picks the star plans for small R).
//
// The binary star cascade materialises I = R |x| S as (a, c) pairs (R
// grouped by B with a counting sort, one prefix sum over S for the output
// positions) and then groups I by A with the same kernel.
#include "mj_kernels.h"

namespace mj {

// slot of `key` in a one-bucket table (the extra slot pool_slots stands for
// key 0xFFFFFFFF), or STAR_NONE
__device__ __forceinline__ uint32_t star_slot(const StarTable& T, uint32_t key) {
    const DirEntry e = T.dir[0];
    if (key == EMPTY_KEY) return e.special ? T.pool_slots : STAR_NONE;
    const uint32_t mask = (1u << e.log2cap) - 1u;
    uint32_t s = slot_hash(key, T.slot_seed) & mask;
    while (true) {
        const uint2 kv = T.pool[e.offset + s];
        if (kv.x == key) return (uint32_t)(e.offset + s);
        if (kv.x == EMPTY_KEY) return STAR_NONE;
        s = (s + 1u) & mask;
    }
}

// id of `key` through R's (key, id) table in global memory, or STAR_NONE
__device__ __forceinline__ uint32_t star_id(const StarTable& R, const uint2* idtab,
                                            const unsigned long long* rid, uint32_t key) {
    const DirEntry e = R.dir[0];
    if (key == EMPTY_KEY) return e.special ? (uint32_t)rid[R.pool_slots] : STAR_NONE;
    const uint32_t mask = (1u << e.log2cap) - 1u;
    uint32_t s = slot_hash(key, R.slot_seed) & mask;
    while (true) {
        const uint2 kv = idtab[e.offset + s];
        if (kv.x == key) return kv.y;
        if (kv.x == EMPTY_KEY) return STAR_NONE;
        s = (s + 1u) & mask;
    }
}

// rows of two key columns; packed [n, 2] rows are read as 8-byte pairs
__device__ __forceinline__ uint2 star_row(const uint32_t* col0, const uint32_t* col1,
                                          int64_t stride, uint64_t i) {
    if (stride == 2 && col1 == col0 + 1 && (reinterpret_cast<uintptr_t>(col0) & 7) == 0)
        return reinterpret_cast<const uint2*>(col0)[i];
    return make_uint2(ld_col(col0, i, stride), ld_col(col1, i, stride));
}

// rows [beg, end) of this workgroup's contiguous chunk
__device__ __forceinline__ void star_chunk(uint64_t n, VGrid vg, uint64_t& beg, uint64_t& end) {
    const uint64_t per = (n + vg.nblk - 1) / vg.nblk;
    beg = uint64_t(vg.bid) * per;
    end = min<uint64_t>(n, beg + per);
}

// STAR_U lookups in a one-bucket table in global memory at once: the
// first-slot loads are in flight together and only colliding keys walk
// further.  `tab` holds (key, value) slots; an absent key gives `none`, key
// 0xFFFFFFFF gives `special`.
#ifndef MJ_STAR_U
#define MJ_STAR_U 4
#endif
constexpr int STAR_U = MJ_STAR_U;   // rows per thread per step
__device__ __forceinline__ void star_lookup4(const DirEntry& e, const uint2* __restrict__ tab,
                                             uint32_t slot_seed, const uint32_t (&key)[STAR_U],
                                             const bool (&live)[STAR_U], uint32_t none,
                                             uint32_t special, uint32_t (&out)[STAR_U]) {
    const uint32_t mask = (1u << e.log2cap) - 1u;
    const uint2* base = tab + e.offset;
    uint32_t s[STAR_U];
    uint2 kv[STAR_U];
#pragma unroll
    for (int u = 0; u < STAR_U; ++u) {
        s[u] = slot_hash(key[u], slot_seed) & mask;
        kv[u] = live[u] && key[u] != EMPTY_KEY ? base[s[u]] : make_uint2(EMPTY_KEY, 0u);
    }
#pragma unroll
    for (int u = 0; u < STAR_U; ++u) {
        if (!live[u]) { out[u] = none; continue; }
        if (key[u] == EMPTY_KEY) { out[u] = special; continue; }
        out[u] = probe_from(base, mask, key[u], kv[u], s[u], none);
    }
}

// LDS copies of the dimension tables: STAR_LDS_SLOTS packed (key, value)
// slots, rebuilt by every workgroup from a table region with a cheaper
// hash than the global tables' (one multiply; a poor spread only lengthens
// probes).  Every table copied holds at most STAR_LDS_SLOTS / 2 keys.
__device__ __forceinline__ uint32_t lds_hash(uint32_t key) {
    uint32_t h = key * 0x9E3779B1u;
    return h ^ (h >> 15);
}

__device__ __forceinline__ void lds_build(uint2* tab, const uint2* region, uint32_t cap) {
    constexpr uint32_t mask = STAR_LDS_SLOTS - 1u;
    for (uint32_t s = threadIdx.x; s < STAR_LDS_SLOTS; s += blockDim.x) tab[s] = make_uint2(EMPTY_KEY, 0u);
    __syncthreads();
    for (uint32_t s = threadIdx.x; s < cap; s += blockDim.x) {
        const uint2 kv = region[s];
        if (kv.x == EMPTY_KEY) continue;
        uint32_t h = lds_hash(kv.x) & mask;
        while (atomicCAS(&tab[h].x, EMPTY_KEY, kv.x) != EMPTY_KEY) h = (h + 1u) & mask;   // keys are distinct
        tab[h].y = kv.y;
    }
}

// STAR_U LDS lookups at once: every row's first slot is read together (a
// hit or an empty slot costs one round trip), collisions walk further.
__device__ __forceinline__ void lds_get4(const uint2* tab, const uint32_t (&key)[STAR_U],
                                         const bool (&live)[STAR_U], uint32_t none, uint32_t special,
                                         uint32_t (&out)[STAR_U]) {
    constexpr uint32_t mask = STAR_LDS_SLOTS - 1u;
    uint32_t h[STAR_U];
    uint2 kv[STAR_U];
#pragma unroll
    for (int u = 0; u < STAR_U; ++u) {
        h[u] = lds_hash(key[u]) & mask;
        kv[u] = tab[h[u]];
    }
#pragma unroll
    for (int u = 0; u < STAR_U; ++u) {
        if (!live[u]) { out[u] = none; continue; }
        if (key[u] == EMPTY_KEY) { out[u] = special; continue; }
        out[u] = probe_from(tab, mask, key[u], kv[u], h[u], none);
    }
}

// The rows of this workgroup's chunk, STAR_U per thread per step, with the
// next step's rows loaded before the current ones are processed.
template <typename F>
__device__ __forceinline__ void star_stream(const uint32_t* col0, const uint32_t* col1, int64_t stride,
                                            uint64_t n, VGrid vg, F&& body) {
    uint64_t beg, end;
    star_chunk(n, vg, beg, end);
    const uint64_t nthr = blockDim.x, step = STAR_U * nthr;
    uint2 cur[STAR_U], nxt[STAR_U];
#pragma unroll
    for (int u = 0; u < STAR_U; ++u) {
        const uint64_t idx = beg + threadIdx.x + u * nthr;
        cur[u] = idx < end ? star_row(col0, col1, stride, idx) : make_uint2(0u, 0u);
    }
    for (uint64_t q = beg + threadIdx.x; q < end; q += step) {
#pragma unroll
        for (int u = 0; u < STAR_U; ++u) {
            const uint64_t idx = q + step + u * nthr;
            nxt[u] = idx < end ? star_row(col0, col1, stride, idx) : make_uint2(0u, 0u);
        }
        uint32_t key[STAR_U], c[STAR_U];
        bool live[STAR_U];
#pragma unroll
        for (int u = 0; u < STAR_U; ++u) {
            live[u] = q + u * nthr < end;
            key[u] = cur[u].x;
            c[u] = cur[u].y;
        }
        body(q, key, c, live);
#pragma unroll
        for (int u = 0; u < STAR_U; ++u) cur[u] = nxt[u];
    }
}

MJ_KERNEL(k_star_occ, 256, StarOccArgs) {
    const uint64_t cursor = *A.cursor;
    for (uint64_t i = vg.bid * (uint64_t)blockDim.x + threadIdx.x; i <= A.R.pool_slots;
         i += (uint64_t)vg.nblk * blockDim.x) {
        uint32_t o;
        if (i == A.R.pool_slots) o = A.R.dir[0].special ? 1u : 0u;
        else o = (i < cursor && A.R.pool[i].x != EMPTY_KEY) ? 1u : 0u;
        A.occ[i] = o;
    }
}

MJ_KERNEL(k_star_ids, 256, StarIdArgs) {
    const uint32_t ps = A.R.pool_slots;
    for (uint64_t i = vg.bid * (uint64_t)blockDim.x + threadIdx.x; i < ps;
         i += (uint64_t)vg.nblk * blockDim.x) {
        const bool occ = A.rid[i + 1] != A.rid[i];
        A.idtab[i] = make_uint2(occ ? A.R.pool[i].x : EMPTY_KEY, occ ? (uint32_t)A.rid[i] : 0u);
    }
}

// Group-by of S = (b, c) rows by B, weight mult_T(c): the star three-way
// join's one pass over the fact relation.
MJ_KERNEL(k_star_group_b, STAR_THREADS, StarGroupArgs) {
    __shared__ uint2 ttab[STAR_LDS_SLOTS];
    __shared__ uint2 rtab[STAR_LDS_SLOTS];
    __shared__ unsigned long long acc[STAR_LDS_SLOTS / 2];
    const DirEntry re = A.R.dir[0];
    const DirEntry te = A.T.dir[0];
    const uint32_t rcap = 1u << re.log2cap, tcap = 1u << te.log2cap;
    const uint32_t k = (uint32_t)A.rid[A.R.pool_slots + 1];
    // both tables (and the k sums) in LDS; uniform over the launch
    const bool lds = rcap <= STAR_LDS_SLOTS && tcap <= STAR_LDS_SLOTS && k <= STAR_LDS_SLOTS / 2;
    const uint32_t rspecial = re.special ? (uint32_t)A.rid[A.R.pool_slots] : STAR_NONE;
    const int nthr = blockDim.x;
    if (lds) {
        lds_build(ttab, A.T.pool + te.offset, tcap);
        lds_build(rtab, A.idtab + re.offset, rcap);
        for (uint32_t i = threadIdx.x; i < k; i += nthr) acc[i] = 0;
    }
    __syncthreads();
    star_stream(A.col0, A.col1, A.stride, A.n, vg,
                [&](uint64_t, const uint32_t (&key)[STAR_U], const uint32_t (&c)[STAR_U],
                    const bool (&live)[STAR_U]) {
        uint32_t w[STAR_U], id[STAR_U];
        bool need[STAR_U];
        if (lds) {
            lds_get4(ttab, c, live, 0u, te.special, w);
#pragma unroll
            for (int u = 0; u < STAR_U; ++u) need[u] = w[u] != 0;
            lds_get4(rtab, key, need, STAR_NONE, rspecial, id);
#pragma unroll
            for (int u = 0; u < STAR_U; ++u)                 // an absent b is not in R
                if (id[u] != STAR_NONE) atomicAdd(&acc[id[u]], (unsigned long long)w[u]);
        } else {
            star_lookup4(te, A.T.pool, A.T.slot_seed, c, live, 0u, te.special, w);
#pragma unroll
            for (int u = 0; u < STAR_U; ++u) need[u] = w[u] != 0;
            star_lookup4(re, A.idtab, A.R.slot_seed, key, need, STAR_NONE, rspecial, id);
#pragma unroll
            for (int u = 0; u < STAR_U; ++u)
                if (id[u] != STAR_NONE) atomicAdd(&A.out[id[u]], (unsigned long long)w[u]);
        }
    });
    __syncthreads();
    if (lds)
        for (uint32_t i = threadIdx.x; i < k; i += nthr)
            A.partial[uint64_t(vg.bid) * STAR_STRIDE + i] = acc[i];
}

// Group-by of (a, c) rows by A value, weight mult_T(c): the star cascade's
// second join.  T's table in LDS when it fits, the sums in LDS while
// a_domain <= STAR_GROUPS.
MJ_KERNEL(k_star_group_a, STAR_THREADS, StarGroupArgs) {
    __shared__ uint2 ttab[STAR_LDS_SLOTS];
    __shared__ unsigned long long acc[STAR_GROUPS];
    const DirEntry te = A.T.dir[0];
    const uint32_t tcap = 1u << te.log2cap;
    const bool tlds = tcap <= STAR_LDS_SLOTS;            // uniform over the launch
    const uint32_t ngroups = A.ngroups_max;
    const bool local = ngroups <= STAR_GROUPS;
    const int nthr = blockDim.x;
    if (tlds) lds_build(ttab, A.T.pool + te.offset, tcap);
    if (local)
        for (uint32_t i = threadIdx.x; i < ngroups; i += nthr) acc[i] = 0;
    __syncthreads();
    star_stream(A.col0, A.col1, A.stride, A.n, vg,
                [&](uint64_t, const uint32_t (&key)[STAR_U], const uint32_t (&c)[STAR_U],
                    const bool (&live)[STAR_U]) {
        uint32_t w[STAR_U];
        if (tlds) lds_get4(ttab, c, live, 0u, te.special, w);
        else star_lookup4(te, A.T.pool, A.T.slot_seed, c, live, 0u, te.special, w);
#pragma unroll
        for (int u = 0; u < STAR_U; ++u) {
            if (w[u] == 0) continue;
            if (key[u] >= ngroups) { atomicExch(A.err, 1u); continue; }
            if (local) atomicAdd(&acc[key[u]], (unsigned long long)w[u]);
            else atomicAdd(&A.out[key[u]], (unsigned long long)w[u]);
        }
    });
    __syncthreads();
    if (local)
        for (uint32_t i = threadIdx.x; i < ngroups; i += nthr)
            A.partial[uint64_t(vg.bid) * STAR_STRIDE + i] = acc[i];
}

// ------------------------------------------- small dimensions (STAR_SMALL)
// A table of at most 4096 distinct keys in 8192 LDS slots in which a lookup
// takes one step whatever the key: a bucket (the top bits of the key's hash)
// holds a displacement d that was chosen so that all its keys fall into free
// slots.  Open addressing at the same load took a wave as many steps as its
// longest chain, 6-8, and the pass over S is bound by the instructions it
// issues.  A bucket that found no displacement is marked STAR_WALK and its
// keys sit at the next free slots (two of its keys with equal slot bits, more
// than 8 keys; about one bucket in a table): a lookup in it walks.
constexpr uint32_t STAR_WALK = 0x8000u;
constexpr int STAR_BKT_KEYS = 8;
constexpr int STAR_TRIES = 16;
static_assert(STAR_SMALL <= STAR_LDS_SLOTS / 2 && STAR_LDS_SLOTS <= STAR_WALK, "a free slot ends every walk");
constexpr uint32_t STAR_FIRST = 256;         // buckets placed before the others
static_assert(STAR_THREADS % STAR_FIRST == 0 && STAR_BKTS <= STAR_FIRST + 2 * STAR_THREADS, "three stages");
static_assert(STAR_LDS_SLOTS == 1u << 13, "13 bits of hash number a slot");
static_assert(STAR_BKTS * 2 <= STAR_LDS_SLOTS, "the bucket lists' heads fit where the values go");

struct StarMap {
    uint32_t* key;                 // [STAR_LDS_SLOTS]
    uint16_t* val;                 // [STAR_LDS_SLOTS]
    uint16_t* disp;                // [STAR_BKTS]
};

__device__ __forceinline__ uint32_t star_hash(uint32_t key) { return key * 0x9E3779B1u; }
__device__ __forceinline__ uint32_t star_bkt(uint32_t h) { return h >> 21; }
static_assert(STAR_BKTS == 1u << 11, "star_bkt takes 11 bits");
__device__ __forceinline__ uint32_t star_home(uint32_t h, uint32_t d) {
    return ((h ^ (h >> 19)) + d) & (STAR_LDS_SLOTS - 1u);
}

// the slot of `key` (not EMPTY_KEY) or an empty slot / another key's slot
__device__ __forceinline__ uint32_t star_walk(const uint32_t* key, uint32_t k, uint32_t s) {
    while (key[s] != k && key[s] != EMPTY_KEY) s = (s + 1u) & (STAR_LDS_SLOTS - 1u);
    return s;
}

struct StarScratch {
    uint32_t* ent;                 // [STAR_LDS_SLOTS] tuple | next slot of the bucket's list << 16
    uint32_t* raw;                 // [STAR_SMALL] the key column
    uint32_t* cls;                 // [STAR_BKT_KEYS + 2] buckets by number of keys
    uint32_t* used;                // [STAR_LDS_SLOTS / 32] slots taken, a bit each
};

// Build M over a key column (EMPTY_KEY left out): val = the lowest tuple with
// the key (TUPLE) or the key's multiplicity; M's arrays are scratch
// until the placement.  The lowest EMPTY_KEY tuple, or their number, goes to
// *special.  A bucket belongs to one lane, which finds its displacement 32 at a
// time in a bitmap of the slots taken: the runs of bits from its keys' home
// slots, combined, have a zero where all of them fit (one displacement at a
// time on the slots themselves took 31 us of a build's 50).  The buckets are
// taken in order of their number of keys: a wave's lanes have the same work,
// and the large ones, which seldom get all their slots while others claim
// theirs, go first and alone.
template <bool TUPLE>
__device__ __forceinline__ void star_map_build(const StarMap& M, const uint32_t* col, int64_t stride, uint32_t n,
                               const StarScratch& X, uint32_t* special) {
    constexpr uint32_t MASK = STAR_LDS_SLOTS - 1u, NIL = 0xFFFFu;
    constexpr int PER = 3;
    const uint32_t t = threadIdx.x;
    uint32_t *const ent = X.ent, *const raw = X.raw;
    uint32_t* head = reinterpret_cast<uint32_t*>(M.val);
    uint32_t* count = reinterpret_cast<uint32_t*>(M.disp);     // 16 bits a bucket
    uint16_t* order = reinterpret_cast<uint16_t*>(M.key);      // buckets, most keys first
    for (uint32_t i = t; i < STAR_BKTS / 2; i += STAR_THREADS) count[i] = 0;
    if (t < STAR_BKT_KEYS + 2) X.cls[t] = 0;
    if (t < STAR_LDS_SLOTS / 32) X.used[t] = 0;
    for (uint32_t i = t; i < STAR_LDS_SLOTS; i += STAR_THREADS) ent[i] = EMPTY_KEY;
    for (uint32_t i = t; i < STAR_BKTS; i += STAR_THREADS) head[i] = NIL;
    for (uint32_t i = t; i < n; i += STAR_THREADS) raw[i] = ld_col(col, i, stride);
    if (t == 0) *special = TUPLE ? STAR_NONE : 0u;
    __syncthreads();
    // the distinct keys: ent[] = the lowest tuple with the key
    for (uint32_t i = t; i < n; i += STAR_THREADS) {
        const uint32_t k = raw[i], h = star_hash(k);
        if (k == EMPTY_KEY) {
            if (TUPLE) atomicMin(special, i);
            else atomicAdd(special, 1u);
            continue;
        }
        // a step of the key's own (odd: it meets every slot): a wave waits for
        // its longest chain, and runs of taken slots make chains long
        for (uint32_t s = h >> 19;; s = (s + (h >> 7 | 1u)) & MASK) {
            const uint32_t o = atomicCAS(&ent[s], EMPTY_KEY, i);
            if (o == EMPTY_KEY) break;
            if (raw[o] == k) { atomicMin(&ent[s], i); break; }
        }
    }
    __syncthreads();
    // lists of a bucket's keys
    for (uint32_t s = t; s < STAR_LDS_SLOTS; s += STAR_THREADS) {
        const uint32_t i = ent[s];
        if (i == EMPTY_KEY) continue;
        const uint32_t b = star_bkt(star_hash(raw[i]));
        ent[s] = i | atomicExch(&head[b], s) << 16;
        atomicAdd(&count[b >> 1], 1u << ((b & 1u) * 16u));
    }
    __syncthreads();
    for (uint32_t b = t; b < STAR_BKTS; b += STAR_THREADS) {
        const uint32_t c = min<uint32_t>(M.disp[b], STAR_BKT_KEYS + 1);
        atomicAdd(&X.cls[c], 1u);
    }
    __syncthreads();
    uint32_t larger = 0;                            // buckets with more keys than t
    if (t < STAR_BKT_KEYS + 2)
        for (uint32_t c = t + 1; c < STAR_BKT_KEYS + 2; ++c) larger += X.cls[c];
    __syncthreads();
    if (t < STAR_BKT_KEYS + 2) X.cls[t] = larger;
    __syncthreads();
    for (uint32_t b = t; b < STAR_BKTS; b += STAR_THREADS) {
        const uint32_t c = min<uint32_t>(M.disp[b], STAR_BKT_KEYS + 1);
        order[atomicAdd(&X.cls[c], 1u)] = (uint16_t)b;
    }
    __syncthreads();
    uint32_t bkt[PER], first[PER], size[PER];
    bool walk[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        // stages of 256, then of 1024 buckets
        const uint32_t p = q == 0 ? t : STAR_FIRST + (q - 1) * STAR_THREADS + t;
        const bool mine = p < (q == 0 ? STAR_FIRST : STAR_BKTS);
        bkt[q] = mine ? order[p] : STAR_NONE;
        first[q] = mine ? head[bkt[q]] : NIL;
        size[q] = mine ? M.disp[bkt[q]] : 0u;
    }
    __syncthreads();
    for (uint32_t i = t; i < STAR_LDS_SLOTS; i += STAR_THREADS) M.key[i] = EMPTY_KEY;
    if (!TUPLE)
        for (uint32_t i = t; i < STAR_LDS_SLOTS / 2; i += STAR_THREADS) reinterpret_cast<uint32_t*>(M.val)[i] = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const uint32_t b = bkt[q];
        // the most keys of a bucket of this wave (its first lane's: the order)
        const int most = (int)min<uint32_t>(wave_read(size[q], 0), STAR_BKT_KEYS);
        const int sz = (int)min<uint32_t>(size[q], STAR_BKT_KEYS);
        uint32_t k[STAR_BKT_KEYS], home[STAR_BKT_KEYS], row[STAR_BKT_KEYS], e = first[q];
#pragma unroll
        for (int j = 0; j < STAR_BKT_KEYS; ++j) {
            if (j >= most) break;
            const uint32_t v = j < sz ? ent[e] : 0u;
            row[j] = v & 0xFFFFu;
            k[j] = raw[row[j]];
            home[j] = star_home(star_hash(k[j]), 0u);
            e = v >> 16;
        }
        walk[q] = size[q] > STAR_BKT_KEYS;          // more keys than fit the registers
#pragma unroll
        for (int j = 1; j < STAR_BKT_KEYS; ++j) {
            if (j >= most) break;
#pragma unroll
            for (int l = 0; l < j; ++l) walk[q] = walk[q] || (j < sz && home[j] == home[l]);
        }
        uint32_t d = 0;
        bool placed = walk[q] || sz == 0;
        for (int tries = 0; !placed; ++tries) {
            if (tries == STAR_TRIES) { walk[q] = true; break; }
            uint32_t taken = 0;
#pragma unroll
            for (int j = 0; j < STAR_BKT_KEYS; ++j) {
                if (j >= most) break;
                const uint32_t s = (home[j] + d) & MASK;
                const uint64_t bits = X.used[s >> 5] | uint64_t(X.used[((s >> 5) + 1u) & (MASK >> 5)]) << 32;
                taken |= j < sz ? (uint32_t)(bits >> (s & 31u)) : 0u;
            }
            if (taken == 0xFFFFFFFFu) { d += 32; continue; }
            const uint32_t at_d = d + (uint32_t)__ffs((int)~taken) - 1u;
            uint32_t lost = 0;                      // keys whose slot another bucket took first
#pragma unroll
            for (int j = 0; j < STAR_BKT_KEYS; ++j) {
                if (j >= most) break;
                const uint32_t s = (home[j] + at_d) & MASK;
                if (j < sz) lost |= (atomicOr(&X.used[s >> 5], 1u << (s & 31u)) >> (s & 31u) & 1u) << j;
            }
            placed = lost == 0;
#pragma unroll
            for (int j = 0; j < STAR_BKT_KEYS; ++j) {
                if (j >= most) break;
                const uint32_t s = (home[j] + at_d) & MASK;
                if (placed) {
                    if (j < sz) {
                        M.key[s] = k[j];
                        if (TUPLE) M.val[s] = (uint16_t)row[j];
                    }
                } else if (j < sz && (lost >> j & 1u) == 0) {
                    atomicAnd(&X.used[s >> 5], ~(1u << (s & 31u)));
                }
            }
            // two buckets that took each other's slots part ways
            d = placed ? at_d : at_d + 1 + (b & 15u);
        }
        if (b != STAR_NONE) M.disp[b] = (uint16_t)((d & MASK) | (walk[q] ? STAR_WALK : 0u));
        if (q + 1 < PER) __syncthreads();
    }
    __syncthreads();                                // no slot is claimed for a bucket any more
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (!walk[q]) continue;
        const uint32_t d = M.disp[bkt[q]] & MASK;
        for (uint32_t e = first[q]; e != NIL;) {
            const uint32_t v = ent[e], i = v & 0xFFFFu, k = raw[i];
            uint32_t s = star_home(star_hash(k), d);
            while (atomicCAS(&M.key[s], EMPTY_KEY, k) != EMPTY_KEY) s = (s + 1u) & MASK;
            if (TUPLE) M.val[s] = (uint16_t)i;
            e = v >> 16;
        }
    }
    __syncthreads();
    if (!TUPLE) {
        // at most STAR_SMALL a key: no carry between a word's two halves
        uint32_t* v2 = reinterpret_cast<uint32_t*>(M.val);
        for (uint32_t i = t; i < n; i += STAR_THREADS) {
            const uint32_t k = raw[i];
            if (k == EMPTY_KEY) continue;
            const uint32_t h = star_hash(k);
            const uint32_t s = star_walk(M.key, k, star_home(h, M.disp[star_bkt(h)]));
            atomicAdd(&v2[s >> 1], 1u << ((s & 1u) * 16u));
        }
        __syncthreads();
    }
}

// U lookups in one table: the displacements, the keys, the values, each for
// all U at once.  An absent key gives `none`, key EMPTY_KEY `special`.
template <int U>
__device__ __forceinline__ void star_get(const StarMap& M, const uint32_t (&key)[U], uint32_t none,
                                         uint32_t special, uint32_t (&out)[U]) {
    uint32_t h[U], d[U], s[U], k[U];
#pragma unroll
    for (int u = 0; u < U; ++u) { h[u] = star_hash(key[u]); d[u] = M.disp[star_bkt(h[u])]; }
#pragma unroll
    for (int u = 0; u < U; ++u) { s[u] = star_home(h[u], d[u]); k[u] = M.key[s[u]]; }
    bool walk = false;
#pragma unroll
    for (int u = 0; u < U; ++u) walk = walk || (k[u] != key[u] && (d[u] & STAR_WALK) != 0);
    if (walk) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k[u] != key[u] && (d[u] & STAR_WALK) != 0) { s[u] = star_walk(M.key, key[u], s[u]); k[u] = M.key[s[u]]; }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) out[u] = M.val[s[u]];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        out[u] = k[u] == key[u] ? out[u] : none;
        out[u] = key[u] == EMPTY_KEY ? special : out[u];
    }
}

// The star three-way join for R and T of at most STAR_SMALL tuples: both
// tables in every workgroup's LDS, its contiguous chunk of S streamed past
// them, mult_T(c) added to the sum of b's first R tuple.  One workgroup per
// CU (157 KB of LDS).  Bound by the instructions of two lookups and an LDS
// add a tuple, close behind it by reading S: 2^26 tuples in 159 us, of which
// 35-40 us build the two tables of 4096 tuples each (in every workgroup, at
// once: one workgroup building them for all would take as long and need
// another launch); 115 us of streaming are 4.7 TB/s.  Open addressing in
// tables made by other kernels: 287 us.
MJ_KERNEL(k_star_stream, STAR_THREADS, StarStreamArgs) {
    __shared__ uint32_t tkey[STAR_LDS_SLOTS];
    __shared__ uint32_t rkey[STAR_LDS_SLOTS];
    __shared__ uint32_t tval[STAR_LDS_SLOTS / 2];
    __shared__ uint32_t rval[STAR_LDS_SLOTS / 2];
    __shared__ unsigned long long acc[STAR_SMALL];
    __shared__ uint16_t tdisp[STAR_BKTS];
    __shared__ uint16_t rdisp[STAR_BKTS];
    __shared__ uint32_t raw[STAR_SMALL];
    __shared__ uint32_t cls[STAR_BKT_KEYS + 2];
    __shared__ uint32_t used[STAR_LDS_SLOTS / 32];
    __shared__ uint32_t s_special[2];
    static_assert(sizeof(acc) >= STAR_LDS_SLOTS * sizeof(uint32_t), "the sums' space holds a build's scratch");
    const uint32_t t = threadIdx.x;
    for (uint64_t i = uint64_t(vg.bid) * STAR_THREADS + t; i < A.nzero; i += uint64_t(vg.nblk) * STAR_THREADS)
        A.count[i] = 0;
    const StarMap TM{tkey, reinterpret_cast<uint16_t*>(tval), tdisp};
    const StarMap RM{rkey, reinterpret_cast<uint16_t*>(rval), rdisp};
    const StarScratch X{reinterpret_cast<uint32_t*>(acc), raw, cls, used};
    star_map_build<false>(TM, A.t0, A.t_stride, A.n_t, X, &s_special[0]);
    star_map_build<true>(RM, A.r1, A.r_stride, A.n_r, X, &s_special[1]);
    const uint32_t tspecial = s_special[0], rspecial = s_special[1];
    if (vg.bid == 0) {
        for (uint32_t i = t; i < A.n_r; i += STAR_THREADS) {
            const uint32_t k[1] = {raw[i]};
            uint32_t o[1];
            star_get<1>(RM, k, 0u, rspecial, o);
            A.rep[i] = o[0];
        }
        if (t < 2) A.rep[A.n_r + t] = 0;
    }
    for (uint32_t i = t; i < A.n_r; i += STAR_THREADS) acc[i] = 0;
    __syncthreads();

    constexpr int U = 2 * STAR_PAIRS;
    constexpr uint32_t STEP = U * STAR_THREADS;
    // chunks of whole steps' alignment, so that a pair of rows is one load
    const uint64_t per = ((A.n_s + vg.nblk - 1) / vg.nblk + 1) & ~uint64_t(1);
    const uint64_t beg = min<uint64_t>(A.n_s, uint64_t(vg.bid) * per), cnt = min<uint64_t>(A.n_s - beg, per);
    const bool packed = A.s_stride == 2 && A.s1 == A.s0 + 1 && (reinterpret_cast<uintptr_t>(A.s0) & 15) == 0;
    auto add = [&](const uint2 (&row)[U], const bool (&live)[U]) {
        uint32_t c[U], b[U], w[U], id[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { b[u] = row[u].x; c[u] = row[u].y; }
        star_get<U>(TM, c, 0u, tspecial, w);
        star_get<U>(RM, b, STAR_NONE, rspecial, id);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (live[u] && w[u] != 0 && id[u] != STAR_NONE) atomicAdd(&acc[id[u]], (unsigned long long)w[u]);
    };
    const uint64_t whole = cnt / STEP;
    uint2 cur[U], nxt[U];
    bool live[U];
#pragma unroll
    for (int u = 0; u < U; ++u) live[u] = true;
    auto load = [&](uint64_t step, uint2 (&row)[U]) {          // a whole step: no bounds to check
        if (packed) {
            const uint4* p = reinterpret_cast<const uint4*>(A.s0 + 2 * (beg + step * STEP)) + t;
#pragma unroll
            for (int j = 0; j < (int)STAR_PAIRS; ++j) {
                const uint4 v = p[j * STAR_THREADS];
                row[2 * j] = make_uint2(v.x, v.y);
                row[2 * j + 1] = make_uint2(v.z, v.w);
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
                row[u] = star_row(A.s0, A.s1, A.s_stride, beg + step * STEP + t + u * STAR_THREADS);
        }
    };
    if (whole) load(0, cur);
    for (uint64_t q = 0; q < whole; ++q) {
        if (q + 1 < whole) load(q + 1, nxt);
        add(cur, live);
#pragma unroll
        for (int u = 0; u < U; ++u) cur[u] = nxt[u];
    }
    if (whole * STEP < cnt) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t i = whole * STEP + t + u * STAR_THREADS;
            live[u] = i < cnt;
            cur[u] = live[u] ? star_row(A.s0, A.s1, A.s_stride, beg + i) : make_uint2(0u, 0u);
        }
        add(cur, live);
    }
    __syncthreads();
    for (uint32_t i = t; i < A.n_r; i += STAR_THREADS) A.partial[uint64_t(vg.bid) * STAR_STRIDE + i] = acc[i];
}

// W per first tuple = the workgroups' sums added up, a block for 64 of them
// (16 rows of threads, each every 16th workgroup), then count[a] += W of the
// R tuples they stand for.  The last block makes every count all ones when an
// A value that joins was out of range.
MJ_KERNEL(k_star_finish, STAR_REDUCE_THREADS, StarFinishArgs) {
    constexpr uint32_t ROWS = STAR_REDUCE_THREADS / 64;
    __shared__ unsigned long long part[ROWS][64];
    __shared__ uint32_t s_bad;
    const uint32_t col = threadIdx.x & 63u, row = threadIdx.x >> 6;
    const uint32_t g0 = vg.bid * 64, g = g0 + col;
    unsigned long long s = 0;
    if (g < A.n_r) {
#pragma unroll 8
        for (uint32_t b = row; b < A.nblocks; b += ROWS) s += A.partial[uint64_t(b) * STAR_STRIDE + g];
    }
    part[row][col] = s;
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    if (row == 0) {
#pragma unroll
        for (uint32_t r = 1; r < ROWS; ++r) s += part[r][col];
        part[0][col] = s;
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < A.n_r; i += STAR_REDUCE_THREADS) {
        const uint32_t e = A.rep[i] - g0;
        if (e >= 64) continue;
        const unsigned long long w = part[0][e];
        if (w == 0) continue;
        const uint32_t a = ld_col(A.r0, i, A.r_stride);
        if (a < A.a_domain) atomicAdd(&A.count[a], w);
        else s_bad = 1;
    }
    __syncthreads();
    uint32_t* ticket = A.rep + A.n_r;
    if (!handoff_last(ticket, vg.nblk, s_bad != 0)) return;
    if ((atomicAdd(ticket, 0u) & 0x80000000u) == 0) return;
    for (uint64_t i = threadIdx.x; i < A.a_domain; i += STAR_REDUCE_THREADS) A.count[i] = ~0ull;
}

// out[g] = sum over blocks of partial[block][g] (LDS modes only): a block
// takes 64 groups, its 16 rows of threads each sum every 16th block's
// partials (64 consecutive groups per load), then the rows are added in LDS.
MJ_KERNEL(k_star_reduce, STAR_REDUCE_THREADS, StarReduceArgs) {
    __shared__ unsigned long long part[STAR_REDUCE_THREADS / 64][64];
    uint32_t ngroups;
    if (A.by_b) {
        // k_star_group_b's rule: otherwise its sums are in A.out already
        const uint32_t k = (uint32_t)A.rid[A.pool_slots + 1];
        const bool lds = (1u << A.rdir[0].log2cap) <= STAR_LDS_SLOTS &&
                         (1u << A.tdir[0].log2cap) <= STAR_LDS_SLOTS && k <= STAR_LDS_SLOTS / 2;
        ngroups = lds ? k : 0u;
    } else {
        ngroups = A.ngroups_max <= STAR_GROUPS ? A.ngroups_max : 0u;
    }
    constexpr uint32_t ROWS = STAR_REDUCE_THREADS / 64;
    const uint32_t col = threadIdx.x & 63u, row = threadIdx.x >> 6;
    for (uint32_t g0 = vg.bid * 64; g0 < ngroups; g0 += vg.nblk * 64) {
        const uint32_t g = g0 + col;
        unsigned long long s = 0;
        if (g < ngroups)
            for (uint32_t b = row; b < A.nblocks; b += ROWS) s += A.partial[uint64_t(b) * STAR_STRIDE + g];
        part[row][col] = s;
        __syncthreads();
        if (row == 0 && g < ngroups) {
            unsigned long long t = 0;
#pragma unroll
            for (uint32_t r = 0; r < ROWS; ++r) t += part[r][col];
            A.out[g] = t;
        }
        __syncthreads();
    }
}

MJ_KERNEL(k_star_count, 256, StarCountArgs) {
    for (uint64_t i = vg.bid * (uint64_t)blockDim.x + threadIdx.x; i < A.n;
         i += (uint64_t)vg.nblk * blockDim.x) {
        const uint2 r = star_row(A.col0, A.col1, A.stride, i);
        const uint32_t sl = star_slot(A.R, r.y);
        if (sl == STAR_NONE) continue;
        const unsigned long long w = A.W[A.rid[sl]];
        if (w == 0) continue;
        if (r.x < A.a_domain) atomicAdd(&A.count[r.x], w);
        else atomicExch(A.err, 1u);
    }
}

// --------------------------------------------------------------- cascade
MJ_KERNEL(k_star_rmult, 256, StarRMultArgs) {
    const StarRIndexArgs& X = A.x;
    const uint32_t ps = X.R.pool_slots;
    for (uint64_t i = vg.bid * (uint64_t)blockDim.x + threadIdx.x; i <= ps;
         i += (uint64_t)vg.nblk * blockDim.x) {
        if (X.rid[i + 1] == X.rid[i]) continue;        // not occupied
        A.mult[X.rid[i]] = i == ps ? X.R.dir[0].special : X.R.pool[i].y;
    }
}

MJ_KERNEL(k_star_rfill, 256, StarRIndexArgs) {
    for (uint64_t i = vg.bid * (uint64_t)blockDim.x + threadIdx.x; i < A.n;
         i += (uint64_t)vg.nblk * blockDim.x) {
        const uint2 r = star_row(A.col0, A.col1, A.stride, i);
        const uint32_t sl = star_slot(A.R, r.y);      // every b of R is in its table
        if (sl == STAR_NONE) continue;                // (unless its pool ran out: reported)
        const unsigned long long id = A.rid[sl];
        const uint32_t k = atomicAdd(&A.rcur[id], 1u);
        A.ra[A.roff[id] + k] = r.x;
    }
}

// Join 1 of the cascade in two passes over S (pairs per tuple, then the
// pairs themselves at prefix-sum positions), R's (key, id) table and the
// group offsets in LDS when they fit.
template <bool WRITE>
__device__ void star_join1(const StarExpandArgs& A, VGrid vg, uint2* rtab, unsigned long long* roffs) {
    const DirEntry re = A.R.dir[0];
    const uint32_t rcap = 1u << re.log2cap;
    const uint32_t k = (uint32_t)A.rid[A.R.pool_slots + 1];
    const bool lds = rcap <= STAR_LDS_SLOTS && k < STAR_STRIDE;   // uniform over the launch
    const uint32_t rspecial = re.special ? (uint32_t)A.rid[A.R.pool_slots] : STAR_NONE;
    if (lds) {
        lds_build(rtab, A.idtab + re.offset, rcap);
        for (uint32_t i = threadIdx.x; i <= k; i += blockDim.x) roffs[i] = A.roff[i];
    }
    __syncthreads();
    const uint64_t nthr = blockDim.x;
    star_stream(A.col0, A.col1, A.stride, A.n, vg,
                [&](uint64_t q, const uint32_t (&key)[STAR_U], const uint32_t (&c)[STAR_U],
                    const bool (&live)[STAR_U]) {
        uint32_t id[STAR_U];
        if (lds) {
            lds_get4(rtab, key, live, STAR_NONE, rspecial, id);
        } else {
#pragma unroll
            for (int u = 0; u < STAR_U; ++u) id[u] = live[u] ? star_id(A.R, A.idtab, A.rid, key[u]) : STAR_NONE;
        }
#pragma unroll
        for (int u = 0; u < STAR_U; ++u) {
            if (!live[u]) continue;
            const uint64_t i = q + u * nthr;
            if (!WRITE) {
                A.icnt[i] = id[u] == STAR_NONE ? 0u
                            : (uint32_t)(lds ? roffs[id[u] + 1] - roffs[id[u]] : A.roff[id[u] + 1] - A.roff[id[u]]);
                continue;
            }
            const unsigned long long o = A.ioff[i], cnt = A.ioff[i + 1] - o;
            if (cnt == 0) continue;
            if (o + cnt > A.i_cap) { atomicExch(A.err, 1u); continue; }   // relations other than planned
            const unsigned long long base = lds ? roffs[id[u]] : A.roff[id[u]];
            for (unsigned long long j = 0; j < cnt; ++j) A.I[o + j] = make_uint2(A.ra[base + j], c[u]);
        }
    });
}

MJ_KERNEL(k_star_icount, STAR_THREADS, StarExpandArgs) {
    __shared__ uint2 rtab[STAR_LDS_SLOTS];
    __shared__ unsigned long long roffs[STAR_STRIDE + 1];
    star_join1<false>(A, vg, rtab, roffs);
}

MJ_KERNEL(k_star_expand, STAR_THREADS, StarExpandArgs) {
    __shared__ uint2 rtab[STAR_LDS_SLOTS];
    __shared__ unsigned long long roffs[STAR_STRIDE + 1];
    star_join1<true>(A, vg, rtab, roffs);
}

}  // namespace mj
