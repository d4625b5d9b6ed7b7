// Distinct count of the linear join's D values per A with Flajolet-Martin
// sketches (the footnotes to Example 1 and to Sec. 4's step list: friends of
// friends of friends per person, a union of large overlapping sets that a
// few bytes per set approximate).
//
// The sketch of a set holds FM_WORDS bitmaps; a value x with hash
// h = mix(x) sets bit (trailing zeros of h >> 4, or 28 when h >> 4 is 0) of
// bitmap h & 15, and the estimate is (16 / 0.77351) 2^(mean lowest zero
// bit).  Sketches merge by OR, so the per-A sketch follows the linear join
// with OR in place of the count's sum and product:
//   Tsk[c] = OR over t(c, d) of bit(d)
//   Wsk[b] = OR over s(b, c) of Tsk[c]
//   sketch[a] = OR over r(a, b) of Wsk[b]
// T and S are grouped by sorting their mixed keys (runs of equal high words
// with a prefix directory, as in the cyclic join); a group of 16 lanes, one a
// word, builds the sketch of a short run, and waves that share the elements
// evenly those of the long ones.  R is partitioned by ranges of A, and one
// workgroup ORs its range's sketches in LDS and writes them with their
// estimates.
#include "mj_kernels.h"

namespace mj {

constexpr int FM_GROUP = FM_WORDS;                // lanes of a sketch: one a word
constexpr int FM_FLIGHT = 8;                      // elements a group has in flight
static_assert(WAVE % FM_GROUP == 0 && FM_WORDS == 16, "a hash's low 4 bits name its bitmap");

// where a hash sets its bit: bitmap << 5 | bit
__device__ __forceinline__ uint32_t fm_code(uint32_t h) {
    const uint32_t rest = h >> 4;
    return (h & 15u) << 5 | (rest ? (uint32_t)__builtin_ctz(rest) : 28u);
}

// (16 / 0.77351) * 2^(sum / 16): exact powers of two times 2^(1/16) taken
// (sum mod 16) times, the same sequence of double multiplications the
// definition's reference uses, so that estimates agree bit for bit
__device__ __forceinline__ double fm_estimate(const uint32_t* sk) {
    bool any = false;
    uint32_t sum = 0;
    for (int j = 0; j < FM_WORDS; ++j) {
        any = any || sk[j] != 0;
        sum += sk[j] == 0xFFFFFFFFu ? 32u : (uint32_t)__builtin_ctz(~sk[j]);
    }
    if (!any) return 0.0;
    double p = 1.0;
    for (uint32_t i = 0; i < sum / 16; ++i) p *= 2.0;
    double f = 1.0;
    for (uint32_t i = 0; i < sum % 16; ++i) f *= 1.0442737824274138;   // 2^(1/16)
    return 16.0 / 0.77351 * p * f;
}

// This lane's word of the sketch of elements [i, i + n) of its group (n may
// differ from group to group; all lanes of the wave call this): elem(i) is
// evaluated by one lane an element, 16 elements of a group at once, and
// word(v, l) gives word l of what the element adds, evaluated by the 16 lanes
// of the group for one element after another, FM_FLIGHT of them in flight.
template <typename Elem, typename Word>
__device__ __forceinline__ uint32_t fm_group_or(uint32_t i, uint32_t n, Elem&& elem, Word&& word) {
    const int lane = lane_id(), l = lane & (FM_GROUP - 1), first = lane - l;
    uint32_t sk = 0;
    for (uint32_t o = 0; __ballot(o < n) != 0; o += FM_GROUP) {
        const uint32_t v = o + l < n ? elem(i + o + l) : FM_NONE;
#pragma unroll
        for (int u = 0; u < FM_GROUP; u += FM_FLIGHT) {
            if (__ballot(o + u < n) == 0) break;
            uint32_t w[FM_FLIGHT];
#pragma unroll
            for (int x = 0; x < FM_FLIGHT; ++x) {
                const uint32_t vx = (uint32_t)__shfl((int)v, first + u + x, WAVE);
                w[x] = vx != FM_NONE ? word(vx, l) : 0u;
            }
#pragma unroll
            for (int x = 0; x < FM_FLIGHT; ++x) sk |= w[x];
        }
    }
    return sk;
}

// The sketches of an index's runs.  Runs of at most FM_SHORT elements: a
// group of 16 lanes each, whose words are one 64-byte line.  (One thread a
// run read and wrote each sketch as four 16-byte pieces, 64 lines an
// instruction, and a wave took as long as its longest run.)  Longer runs are
// cleared here and added up by fm_long.
// 4 x 10^6 power-law elements: S's sketches 275 -> 183 us (short and long
// together; random 64-byte reads of T's 16 MB of sketches), T's 89 -> 47 us.
// Uncapped hubs: the long runs 6.5 ms -> 113 us.
template <typename Elem, typename Word>
__device__ __forceinline__ void fm_short(const RunIndex& X, uint32_t* sketch, Elem&& elem, Word&& word) {
    const uint64_t nruns = *X.nruns;
    constexpr uint32_t PER = WAVE / FM_GROUP;
    const int lane = lane_id(), l = lane & (FM_GROUP - 1);
    const uint64_t nw = uint64_t(gridDim.x) * (FM_THREADS / WAVE);
    for (uint64_t r0 = (blockIdx.x * uint64_t(FM_THREADS / WAVE) + threadIdx.x / WAVE) * PER; r0 < nruns;
         r0 += nw * PER) {
        const uint64_t r = r0 + lane / FM_GROUP;
        const bool mine = r < nruns;
        const uint32_t b = mine ? X.run_start[r] : 0u, n = mine ? X.run_start[r + 1] - b : 0u;
        const uint32_t sk = fm_group_or(b, n > FM_SHORT ? 0u : n, elem, word);
        if (mine) sketch[r * FM_WORDS + l] = sk;
    }
}

// The longer runs, a wave for FM_TILE elements of the whole array whatever
// runs they belong to (a hub's run is shared by many waves): their parts of
// long runs are ORed into the cleared sketches.
template <typename Elem, typename Word>
__device__ __forceinline__ void fm_long(const RunIndex& X, uint32_t* sketch, Elem&& elem, Word&& word) {
    const uint64_t nruns = *X.nruns;
    if (nruns == 0) return;
    const uint32_t n = X.run_start[nruns];
    const int lane = lane_id(), l = lane & (FM_GROUP - 1), g = lane / FM_GROUP;
    constexpr uint32_t PER = WAVE / FM_GROUP;
    const uint64_t nw = uint64_t(gridDim.x) * (FM_THREADS / WAVE);
    for (uint64_t t = blockIdx.x * uint64_t(FM_THREADS / WAVE) + threadIdx.x / WAVE; t * FM_TILE < n; t += nw) {
        const uint32_t lo = (uint32_t)(t * FM_TILE), hi = (uint32_t)min<uint64_t>(n, uint64_t(lo) + FM_TILE);
        uint64_t ra = 0, rb = nruns;                       // the run of element lo: the last that starts at or before it
        while (rb - ra > 1) {                              // a lane a candidate
            const uint64_t step = (rb - ra + WAVE - 1) / WAVE, m = ra + lane * step;
            const int c = __popcll(__ballot(m < rb && X.run_start[m] <= lo));        // at least lane 0
            ra += (c - 1) * step;
            rb = min<uint64_t>(rb, ra + step);
        }
        for (uint64_t r0 = ra; r0 < nruns; r0 += WAVE) {
            const uint64_t r = r0 + lane;
            const uint32_t b = r < nruns ? X.run_start[r] : n, e = r < nruns ? X.run_start[r + 1] : n;
            for (uint64_t m = __ballot(b < hi && e - b > FM_SHORT); m; m &= m - 1) {
                const int j = __ffsll((unsigned long long)m) - 1;
                const uint32_t pb = max(wave_read(b, j), lo), pe = min(wave_read(e, j), hi);
                const uint32_t per = (pe - pb + PER - 1) / PER;          // a group's share
                const uint32_t gb = min(pe, pb + g * per);
                uint32_t sk = fm_group_or(gb, min(pe, gb + per) - gb, elem, word);
                sk |= (uint32_t)__shfl_xor((int)sk, 16, WAVE);
                sk |= (uint32_t)__shfl_xor((int)sk, 32, WAVE);
                if (g == 0 && sk) atomicOr(sketch + (r0 + j) * FM_WORDS + l, sk);
            }
            if (wave_read(e, WAVE - 1) >= hi) break;
        }
    }
}

__global__ void __launch_bounds__(FM_THREADS)
k_fm_tsketch(FmTArgs A) {
    fm_short(A.T, A.tsk, [&](uint32_t i) { return fm_code((uint32_t)A.Tk[i]); },
             [](uint32_t c, int l) { return c >> 5 == (uint32_t)l ? 1u << (c & 31u) : 0u; });
}

__global__ void __launch_bounds__(FM_THREADS)
k_fm_tsketch_long(FmTArgs A) {
    fm_long(A.T, A.tsk, [&](uint32_t i) { return fm_code((uint32_t)A.Tk[i]); },
            [](uint32_t c, int l) { return c >> 5 == (uint32_t)l ? 1u << (c & 31u) : 0u; });
}

__global__ void __launch_bounds__(FM_THREADS)
k_fm_wsketch(FmWArgs A) {
    fm_short(A.S, A.wsk, [&](uint32_t i) { return run_find(A.T, (uint32_t)A.Sk[i]); },
             [&](uint32_t t, int l) { return A.tsk[uint64_t(t) * FM_WORDS + l]; });
}

__global__ void __launch_bounds__(FM_THREADS)
k_fm_wsketch_long(FmWArgs A) {
    fm_long(A.S, A.wsk, [&](uint32_t i) { return run_find(A.T, (uint32_t)A.Sk[i]); },
            [&](uint32_t t, int l) { return A.tsk[uint64_t(t) * FM_WORDS + l]; });
}

// The sketches of ranges that are split into pieces.
__global__ void __launch_bounds__(FM_A_THREADS)
k_fm_clear(FmAArgs A) {
    const uint32_t k = blockIdx.x;
    if (split_pieces(A.rstarts[k + 1] - A.rstarts[k], A.split.chunk) == 1) return;
    const uint64_t lo = uint64_t(k) << A.a_shift, hi = min<uint64_t>(A.a_domain, lo + (uint64_t(1) << A.a_shift));
    for (uint64_t i = lo * FM_WORDS + threadIdx.x; i < hi * FM_WORDS; i += FM_A_THREADS) A.sketch[i] = 0;
}

// One workgroup per range of A, or several when R's A values are skewed (a
// range of 10^6 tuples kept one busy for 3.9 ms), its sketches in LDS.  A lane looks up its R
// tuple's run of S; then the 16 lanes of a group add the words of one tuple
// after another, so that a sketch is read as one line and the words of a
// wave's four tuples lie in 64 consecutive words of LDS each in their own
// banks (a thread a tuple met 4 banks an instruction).  4 x 10^6 tuples:
// 270 -> 190 us, bound by the random reads of S's sketches from beyond L2;
// more reads in flight change nothing.
template <uint32_t SHIFT>
__device__ __forceinline__ void fm_ranges_or(const FmAArgs& A) {
    __shared__ uint32_t acc[(1u << SHIFT) * FM_WORDS];
    if (blockIdx.x >= *A.split.nitems) return;
    const uint32_t item = A.split.items[blockIdx.x], k = item & 0xFFFu, piece = item >> 12;
    const uint64_t base = uint64_t(k) << A.a_shift;
    // ranges past a_domain only receive keys out of range (reported)
    const uint32_t span = base < A.a_domain
                              ? (uint32_t)min<uint64_t>(uint64_t(1) << A.a_shift, A.a_domain - base) : 0u;
    for (uint32_t i = threadIdx.x; i < span * FM_WORDS; i += FM_A_THREADS) acc[i] = 0;
    __syncthreads();
    const int lane = lane_id(), l = lane & (FM_GROUP - 1), first = lane - l;
    const uint32_t s0 = A.rstarts[k], len = A.rstarts[k + 1] - s0, pcs = split_pieces(len, A.split.chunk);
    const uint32_t qb = s0 + (uint32_t)(uint64_t(len) * piece / pcs);
    const uint32_t qe = s0 + (uint32_t)(uint64_t(len) * (piece + 1) / pcs);
    for (uint32_t q0 = qb + (threadIdx.x - lane); q0 < qe; q0 += FM_A_THREADS) {     // uniform over a wave
        const uint32_t q = q0 + lane;
        uint32_t w = FM_NONE, off = 0;
        if (q < qe) {
            const uint2 r = A.R[q];
            const uint64_t o = uint64_t(r.x) - base;
            if (r.x >= A.a_domain || o >= span) atomicExch(A.err, 1u);
            else { off = (uint32_t)o; w = run_find(A.S, mix32(r.y, A.seed)); }       // b's run in S, if any
        }
#pragma unroll
        for (int u = 0; u < FM_GROUP; u += FM_FLIGHT) {
            uint32_t v[FM_FLIGHT], at[FM_FLIGHT];
#pragma unroll
            for (int x = 0; x < FM_FLIGHT; ++x) {
                const uint32_t wx = (uint32_t)__shfl((int)w, first + u + x, WAVE);
                at[x] = (uint32_t)__shfl((int)off, first + u + x, WAVE);
                v[x] = wx != FM_NONE ? A.wsk[uint64_t(wx) * FM_WORDS + l] : 0u;
            }
#pragma unroll
            for (int x = 0; x < FM_FLIGHT; ++x)
                if (v[x]) atomicOr(&acc[at[x] * FM_WORDS + l], v[x]);
        }
    }
    __syncthreads();
    uint32_t* out = A.sketch + base * FM_WORDS;
    if (pcs > 1) {                                        // cleared by k_fm_clear; the last piece has the range's ORs
        for (uint32_t i = threadIdx.x; i < span * FM_WORDS; i += FM_A_THREADS)
            if (acc[i]) atomicOr(&out[i], acc[i]);
        if (!handoff_last(&A.split.done[k], pcs)) return;
        if (threadIdx.x == 0) A.split.done[k] = 0;
        if (!A.est) return;
        for (uint32_t i = threadIdx.x; i < span * FM_WORDS; i += FM_A_THREADS) acc[i] = out[i];
        __syncthreads();
    } else {
        for (uint32_t i = threadIdx.x; i < span * FM_WORDS; i += FM_A_THREADS) out[i] = acc[i];
    }
    if (A.est)
        for (uint32_t i = threadIdx.x; i < span; i += FM_A_THREADS) A.est[base + i] = fm_estimate(acc + i * FM_WORDS);
}

__global__ void __launch_bounds__(FM_A_THREADS)
k_fm_asketch(FmAArgs A) { fm_ranges_or<FM_RANGE_SHIFT>(A); }
__global__ void __launch_bounds__(FM_A_THREADS)
k_fm_asketch_wide(FmAArgs A) { fm_ranges_or<FM_RANGE_MAX_SHIFT>(A); }

__global__ void k_fm_asketch_global(FmAArgs A) {
    for (uint64_t q = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; q < A.n;
         q += (uint64_t)gridDim.x * blockDim.x) {
        const uint2 r = A.R[q];
        if (r.x >= A.a_domain) { atomicExch(A.err, 1u); continue; }
        const uint32_t w = run_find(A.S, mix32(r.y, A.seed));
        if (w == FM_NONE) continue;
        for (int j = 0; j < FM_WORDS; ++j) {
            const uint32_t v = A.wsk[uint64_t(w) * FM_WORDS + j];
            if (v) atomicOr(A.sketch + uint64_t(r.x) * FM_WORDS + j, v);
        }
    }
}

__global__ void k_fm_estimate(FmAArgs A) {
    if (!A.est) return;
    for (uint64_t a = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; a < A.a_domain;
         a += (uint64_t)gridDim.x * blockDim.x)
        A.est[a] = fm_estimate(A.sketch + a * FM_WORDS);
}

}  // namespace mj
