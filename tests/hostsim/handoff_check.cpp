// Host-build check of the table builds' hand-off (test infrastructure only):
// the last piece of a split bucket finds the other pieces' rows and counts as
// they were before the kernel, as if their write-back had not arrived.  What
// it then reads is not the join's, but every access has to stay inside the
// buffers (exact-size allocations under the sanitizers), whatever a count
// left in memory says.
#include <cstdio>
#include <random>
#include <vector>

#include "mj_kernels.h"

using namespace mj;

namespace {

constexpr uint32_t PIECES = 3, CHUNK = SPLIT_MIN_CHUNK, N = PIECES * CHUNK;

struct Split {                        // one bucket of N tuples, its last piece the only one that runs
    std::vector<uint32_t> items{(PIECES - 1) << 12}, nitems{1}, hrow{0}, done{PIECES - 1};
    BucketItems view() { return BucketItems{items.data(), nitems.data(), hrow.data(), done.data(), CHUNK}; }
};

void table(uint32_t stale_count, uint32_t stale_key_range) {
    std::mt19937 g(7);
    std::vector<uint32_t> keys(N), starts{0, N}, err(1), row_special(PIECES, 0), row_n(PIECES, stale_count);
    for (auto& k : keys) k = g() % 300;
    std::vector<uint2> rows(PIECES * DB_CAP), pool(4 * N + 2 * DB_MIN_CAP);
    for (auto& r : rows) r = make_uint2(g() % stale_key_range, 1 + g() % 9);
    std::vector<DirEntry> dir(1);
    std::vector<unsigned long long> cursor{DB_MIN_CAP};
    Split sp;
    DBuildArgs D{};
    D.keys = keys.data(); D.starts = starts.data(); D.nbkt = 1; D.slot_seed = 11;
    D.dir = dir.data(); D.pool = pool.data(); D.pool_cursor = cursor.data(); D.pool_cap = pool.size();
    D.err = err.data(); D.split = sp.view();
    D.rows = rows.data(); D.row_special = row_special.data(); D.row_n = row_n.data();
    hipLaunchKernelGGL(k_dbuild, dim3(1), dim3(DB_THREADS), 0, nullptr, D);
    std::printf("[handoff] k_dbuild, counts of %u, keys below %u: no access out of bounds\n", stale_count,
                stale_key_range);
}

void wtable(uint32_t stale_count, uint32_t stale_key_range) {
    std::mt19937 g(8);
    std::vector<uint2> S(N);
    for (auto& s : S) s = make_uint2(g() % 300, g() % 50);
    std::vector<uint32_t> sstarts{0, N}, err(1), row_n(PIECES, stale_count);
    std::vector<uint2> dpool(128, make_uint2(EMPTY_KEY, 0));           // T's one table: C values 0..49, twice each
    for (uint32_t c = 0; c < 50; ++c) {
        uint32_t s = slot_hash(c, 13) & 127u;
        while (dpool[s].x != EMPTY_KEY) s = (s + 1) & 127u;
        dpool[s] = make_uint2(c, 2);
    }
    std::vector<DirEntry> ddir{DirEntry{0, 7, 0}};
    std::vector<WSlot> rows(PIECES * CELL_CAP), wpool(4 * N + 2 * W_MIN_CAP);
    for (auto& r : rows) r = WSlot{(uint32_t)(g() % stale_key_range), 0, 1ull + g() % 9};
    std::vector<unsigned long long> row_special(PIECES, 0), wcursor{W_MIN_CAP};
    std::vector<WDirEntry> wdir(1);
    Split sp;
    WBuildArgs W{};
    W.S = S.data(); W.sstarts = sstarts.data(); W.ddir = ddir.data(); W.dpool = dpool.data();
    W.c_seed = 1; W.c_bits = 0; W.slot_seed = 13; W.w_seed = 17;
    W.wdir = wdir.data(); W.wpool = wpool.data(); W.wcursor = wcursor.data(); W.wcap = wpool.size();
    W.err = err.data(); W.split = sp.view();
    W.rows = rows.data(); W.row_special = row_special.data(); W.row_n = row_n.data();
    hipLaunchKernelGGL(k_wbuild, dim3(1), dim3(CELL_THREADS), 0, nullptr, W);
    std::printf("[handoff] k_wbuild, counts of %u, keys below %u: no access out of bounds\n", stale_count,
                stale_key_range);
}

}  // namespace

int main() {
    // a count one past a row, a bucket's worth (what a histogram holds), any word;
    // keys that fit the table, and more of them than it takes
    for (uint32_t keys : {500u, 1u << 30})
        for (uint32_t count : {DB_CAP + 1, 1u << 20, 0xFFFFFFFFu}) {
            table(count, keys);
            wtable(count, keys);
        }
    std::printf("[handoff] all checks passed\n");
    return 0;
}
