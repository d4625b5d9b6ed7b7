// Stable LSD radix sort of 64-bit keys (8-bit digits), the repeated radix
// partitioning that groups each relation of the cyclic join by its join key
// (Fig. 3 partitions by radix digits of A, B and C).  Up to RS_MAX_JOBS
// arrays are sorted by the same launches, and the first pass makes the keys
// from the relations' columns, so no unsorted key array is written.
//
//   k_rs_hist    : per tile, digit histogram -> column `tile` of hist[d][tile]
//   (k_part_rowscan: each digit's prefix over tiles and its total; with at
//   most RS_SELF_TILES tiles the scatter adds up the rows itself)
//   k_rs_scatter : per tile, stable ranks, the tile put in digit order in LDS
//                  and written out, each digit's run consecutive
//   k_rs_small   : arrays of at most RS_SMALL keys are sorted whole in one
//                  workgroup's LDS, in one launch.
#include "mj_kernels.h"

namespace mj {

// key i of a job: (mix(key) << 32 | mix(other)), or the other value itself as
// low word, from the columns on the first pass; the stored key afterwards
__device__ __forceinline__ unsigned long long rs_key(const RsJob& J, uint64_t i) {
    if (!J.key_col) return J.in[i];
    const uint32_t hi = ld_col(J.key_col, i, J.stride);
    const uint32_t lo = ld_col(J.val_col, i, J.stride);
    return ((unsigned long long)mix32(hi, J.seed) << 32) | (J.raw_low ? lo : mix32(lo, J.seed));
}

// Keys i0, i0 + step, ... (N of them; past the end the last one again), all
// their loads in flight at once: with a load and its mix key by key, a tile
// of the first pass took eight times the memory's latency.
template <int N>
__device__ __forceinline__ void rs_keys(const RsJob& J, uint64_t i0, uint32_t step, unsigned long long (&key)[N]) {
    const uint64_t last = J.n - 1;
    if (!J.key_col) {
#pragma unroll
        for (int k = 0; k < N; ++k) key[k] = J.in[min<uint64_t>(i0 + uint64_t(k) * step, last)];
        return;
    }
    const uint32_t *kc = J.key_col, *vc = J.val_col;
    const int64_t stride = J.stride;
    uint32_t hi[N], lo[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const uint64_t i = min<uint64_t>(i0 + uint64_t(k) * step, last);
        hi[k] = ld_col(kc, i, stride);
        lo[k] = ld_col(vc, i, stride);
    }
    const uint32_t seed = J.seed;
    const bool raw = J.raw_low != 0;
#pragma unroll
    for (int k = 0; k < N; ++k)
        key[k] = ((unsigned long long)mix32(hi[k], seed) << 32) | (raw ? lo[k] : mix32(lo[k], seed));
}

__device__ __forceinline__ int rs_find_job(const RsLaunch& L, uint32_t tile) {
    int j = 0;
#pragma unroll
    for (int q = 1; q < RS_MAX_JOBS; ++q)
        if (q < L.njobs && tile >= L.job[q].tile_begin) j = q;
    return j;
}

// Bound by reading the keys: 2^26 random ones 109 us a pass, 4.9 TB/s.  With
// all loads of a tile in flight and one add a run of digits the eight passes
// of a general join of 10^6 tuples take 98 us, 188 before.
MJ_KERNEL(k_rs_hist, RS_THREADS, RsLaunch) {
    __shared__ uint32_t lh[256];
    const uint32_t blk = xcd_remap(vg.bid, vg.nblk);
    const RsJob& J = A.job[rs_find_job(A, blk)];
    const uint32_t tile = blk - J.tile_begin;
    for (uint32_t d = threadIdx.x; d < 256; d += blockDim.x) lh[d] = 0;
    __syncthreads();
    const uint64_t beg = uint64_t(tile) * RS_TILE;
    constexpr int ITEMS = RS_TILE / RS_THREADS;
    unsigned long long key[ITEMS];
    rs_keys<ITEMS>(J, beg + threadIdx.x, RS_THREADS, key);
    // one add per run of equal digits of a wave: later passes meet the runs of
    // equal keys that earlier ones made, and adds to one address take turns
    const int lane = lane_id();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const bool live = beg + k * RS_THREADS + threadIdx.x < J.n;
        const uint32_t d = live ? (uint32_t)(key[k] >> A.shift) & 255u : 256u;
        const uint32_t up = __shfl_up(d, 1, WAVE);
        const bool head = lane == 0 || d != up;
        const unsigned long long after = (__ballot(head) >> lane) >> 1;
        if (head && live) atomicAdd(&lh[d], after ? (uint32_t)__ffsll(after) : (uint32_t)(WAVE - lane));
    }
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < 256; d += blockDim.x) J.hist[uint64_t(d) * J.ntiles + tile] = lh[d];
}

// exclusive prefix over the first 256 threads' values (four waves; all
// threads of the workgroup call it, the others' results are unused)
__device__ __forceinline__ uint32_t rs_scan256(uint32_t v, uint32_t* wsum) {
    const int lane = lane_id();
    const uint32_t w = threadIdx.x / WAVE, x = v;
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1) {
        const uint32_t y = __shfl_up(v, off, WAVE);
        if (lane >= off) v += y;
    }
    if (lane == WAVE - 1) wsum[w] = v;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t q = 0; q < w && q < 4; ++q) before += wsum[q];
    __syncthreads();
    return before + v - x;
}

// A tile's keys stay in registers: wave w holds the tile's w-th part in input
// order, 64 keys a round.  The rank of a key among the wave's equal digits is
// the count of earlier rounds (an LDS counter per wave and digit) plus its
// position among the round's matching lanes (eight ballots), so the rounds
// need no barrier; the waves' counters are then added up per digit.  Writing
// from the LDS stage, a digit's run is consecutive (about 16 keys, 128 bytes):
// stores straight from registers are one L2 request a key.  Bound by HBM
// traffic for large arrays (2^26 keys: 478 -> 310 us a pass against
// the unstaged form with five barriers per 256 keys) and by the launch for
// arrays of up to about 10^6.
MJ_KERNEL(k_rs_scatter, RS_THREADS, RsLaunch) {
    constexpr int NW = RS_THREADS / WAVE, ROUNDS = RS_TILE / RS_THREADS;
    __shared__ unsigned long long stage[RS_TILE];
    __shared__ uint16_t wcnt[NW][256];
    __shared__ uint32_t lstart[256], gbase[256];
    __shared__ uint32_t wsum[NW];
    // adjacent tiles write adjacent runs of every digit: keep them on one XCD
    const uint32_t blk = xcd_remap(vg.bid, vg.nblk);
    const RsJob& J = A.job[rs_find_job(A, blk)];
    const uint32_t tile = blk - J.tile_begin;
    const uint32_t lane = lane_id(), w = threadIdx.x / WAVE;
    const uint64_t beg = uint64_t(tile) * RS_TILE;
    const uint32_t cnt = (uint32_t)min<uint64_t>(RS_TILE, J.n - beg);
    const uint32_t at = w * (RS_TILE / NW) + lane;
    unsigned long long key[ROUNDS];
    rs_keys<ROUNDS>(J, beg + at, WAVE, key);
    for (uint32_t d = lane; d < 256; d += WAVE) wcnt[w][d] = 0;
    // digit totals before this tile, and over all tiles
    uint32_t pre = 0, tot = 0;
    if (threadIdx.x < 256) {
        const uint32_t* row = J.hist + uint64_t(threadIdx.x) * J.ntiles;
        if (A.rows) {
            pre = row[tile];
            tot = J.counts[threadIdx.x];
        } else {
            for (uint32_t t = 0; t < J.ntiles; ++t) {
                const uint32_t c = row[t];
                pre += t < tile ? c : 0u;
                tot += c;
            }
        }
    }
    const unsigned long long lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    uint16_t rank[ROUNDS];
#pragma unroll
    for (int k = 0; k < ROUNDS; ++k) {
        wave_fence();
        const bool live = at + k * WAVE < cnt;
        const uint32_t d = (uint32_t)(key[k] >> A.shift) & 255u;
        unsigned long long peers = __ballot(live);          // lanes holding the same digit
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const unsigned long long bal = __ballot(live && ((d >> bit) & 1u));
            peers &= ((d >> bit) & 1u) ? bal : ~bal;
        }
        const uint32_t mine = __popcll(peers & lt_mask);
        const uint32_t before = wcnt[w][d];
        rank[k] = (uint16_t)(before + mine);
        wave_fence();
        if (live && mine == 0) wcnt[w][d] = (uint16_t)(before + __popcll(peers));
    }
    __syncthreads();
    uint32_t local = 0;
    if (threadIdx.x < 256)
        for (int q = 0; q < NW; ++q) {
            const uint32_t c = wcnt[q][threadIdx.x];
            wcnt[q][threadIdx.x] = (uint16_t)local;
            local += c;
        }
    const uint32_t ls = rs_scan256(local, wsum);
    const uint32_t gs = rs_scan256(tot, wsum);
    if (threadIdx.x < 256) {
        lstart[threadIdx.x] = ls;
        gbase[threadIdx.x] = gs + pre - ls;                 // (modulo 2^32)
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ROUNDS; ++k) {
        if (at + k * WAVE >= cnt) continue;
        const uint32_t d = (uint32_t)(key[k] >> A.shift) & 255u;
        stage[lstart[d] + wcnt[w][d] + rank[k]] = key[k];
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < cnt; i += RS_THREADS) {
        const unsigned long long v = stage[i];
        J.out[(uint32_t)(gbase[(uint32_t)(v >> A.shift) & 255u] + i)] = v;
    }
}

// The keys ordered on their bits from `shift` up, ties in input order: the
// order the passes from `shift` up produce.  With shift = 0 the keys are
// sorted as they are (equal keys cannot be told apart).  Otherwise each key's
// digits are packed above its index, which makes every composite distinct,
// the composites are sorted, and each position takes the key its index names
// (kept in LDS beside them).  A bitonic network over the next power of two,
// padded with the largest value; pads sort after every real entry.
// One workgroup per job.
MJ_KERNEL(k_rs_small, RS_SMALL_THREADS, RsLaunch) {
    const RsJob& J = A.job[vg.bid];
    unsigned long long* keys = J.out;
    const uint32_t n = (uint32_t)J.n, shift = A.shift;
    extern __shared__ unsigned long long rs_lds[];
    uint32_t P = 2;
    while (P < n) P <<= 1;
    unsigned long long* v = rs_lds;
    // sorting on the bits above `shift` only: the sort key is those bits
    // with the element's index below them, so equal keys keep their order
    for (uint32_t i = threadIdx.x; i < P; i += blockDim.x) {
        unsigned long long x = ~0ull;
        if (i < n) {
            const unsigned long long k = rs_key(J, i);
            if (shift && J.key_col) keys[i] = k;            // gathered again below
            x = shift ? (((k >> shift) << RS_SMALL_BITS) | i) : k;
        }
        v[i] = x;
    }
    __syncthreads();
    for (uint32_t k = 2; k <= P; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            for (uint32_t t = threadIdx.x; t < P / 2; t += blockDim.x) {
                const uint32_t lo = 2 * t - (t & (j - 1));   // t with a 0 bit inserted at j
                const uint32_t hi = lo + j;
                const unsigned long long a = v[lo], b = v[hi];
                if ((a > b) == ((lo & k) == 0)) {
                    v[lo] = b;
                    v[hi] = a;
                }
            }
            __syncthreads();
        }
    }
    if (shift) {                      // the original keys, in sorted order, gathered before any is overwritten
        for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) v[i] = keys[uint32_t(v[i]) & (RS_SMALL - 1u)];
        __syncthreads();
    }
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) keys[i] = v[i];
}

}  // namespace mj
