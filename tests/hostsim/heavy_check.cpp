// Host-build check of the cyclic join's heavy work items (test infrastructure
// only) at sizes no test can fill with data: a join value with 2^27 tuples on
// both sides has 2^16 x 2^16 = 2^32 items, one more than 32 bits count.  The
// run indexes are made up; the lists lie in sparse mappings of which only the
// part that the last item reads is written.
#include <sys/mman.h>

#include <cstdio>
#include <cstdlib>
#include <type_traits>
#include <vector>

#include "mj_kernels.h"

using namespace mj;

namespace {

int fails = 0;
void expect(bool ok, const char* what, unsigned long long got, unsigned long long want) {
    std::printf("[heavy] %-52s %s (%llu, expected %llu)\n", what, ok ? "ok" : "FAILED", got, want);
    if (!ok) ++fails;
}

uint32_t* sparse(uint64_t words) {
    void* p = mmap(nullptr, words * 4, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED) { std::perror("mmap"); std::exit(2); }
    return static_cast<uint32_t*>(p);
}

// one run of `len` words under `key`
struct OneRun {
    std::vector<uint32_t> key, start, dir{0, 1};
    unsigned long long nruns = 1;
    OneRun(uint32_t k, uint32_t len) : key{k}, start{0, len} {}
    RunIndex view() { return RunIndex{key.data(), start.data(), dir.data(), 0, &nruns}; }
};

void classify(uint32_t x, uint32_t gn, uint64_t want) {
    OneRun stg(9, x), grp(9, gn);
    std::vector<uint2> light(1);
    std::vector<uint32_t> group(1, 77);
    std::vector<unsigned long long> off(1, 77);
    uint32_t nlight = 0;
    unsigned long long heavy = 0;
    TriClassifyPair C{};
    for (int q = 0; q < 2; ++q) {
        C.pass[q].Stg = stg.view(); C.pass[q].Grp = grp.view();
        C.pass[q].share = 1; C.pass[q].nlight = &nlight; C.pass[q].light = light.data();
        C.pass[q].heavy = &heavy; C.pass[q].heavy_group = group.data(); C.pass[q].heavy_off = off.data();
    }
    C.per = 1;
    hipLaunchKernelGGL(k_tri_classify, dim3(1), dim3(256), 0, nullptr, C);       // pass 0 alone
    const unsigned long long items = heavy & ((1ull << HEAVY_SHIFT) - 1ull);
    expect(heavy >> HEAVY_SHIFT == 1 && items == want && group[0] == 0 && off[0] == 0, "items of one heavy group", items,
           want);
}

// the last item alone: the queue's counter stands before it
void last_item() {
    const uint32_t n = 1u << 27;
    OneRun stg(9, n), grp(9, n), itr(5, 3);
    uint32_t *stgl = sparse(n), *grpl = sparse(n);
    for (uint32_t q = 0; q < TRI_HEAVY_X; ++q) stgl[n - TRI_HEAVY_X + q] = 1 + q;
    for (uint32_t q = 0; q < TRI_HEAVY_S; ++q) grpl[n - TRI_HEAVY_S + q] = 5;    // each s meets the list below
    std::vector<uint32_t> itrl{7, TRI_HEAVY_X, TRI_HEAVY_X + 9};                  // two of its entries are staged
    unsigned long long total = 0, heavy = (1ull << HEAVY_SHIFT) | (1ull << 32);
    std::vector<uint32_t> group(1, 0);
    std::vector<unsigned long long> off(1, 0);
    std::remove_pointer<decltype(TriJoinArgs::heavy_next)>::type next = 0xFFFFFFFFu, done = 0;
    unsigned long long none = 0;
    uint32_t zero = 0;
    TriJoinPair J{};
    for (int q = 0; q < 2; ++q) {
        J.pass[q].Stg = stg.view(); J.pass[q].Grp = grp.view(); J.pass[q].Itr = itr.view();
        J.pass[q].Stgl = stgl; J.pass[q].Grpl = grpl; J.pass[q].Itrl = itrl.data();
        J.pass[q].strict = 1; J.pass[q].nlight = &zero; J.pass[q].heavy = q ? &none : &heavy;
        J.pass[q].heavy_group = group.data(); J.pass[q].heavy_off = off.data();
        J.pass[q].heavy_next = q ? &done : &next; J.pass[q].share = 1; J.pass[q].low_bits = 0; J.pass[q].total = &total;
    }
    hipLaunchKernelGGL(k_tri_heavy, dim3(1), dim3(TRI_HEAVY_THREADS), 0, nullptr, J);
    expect(total == 2ull * TRI_HEAVY_S, "matches of the last of 2^32 items", total, 2ull * TRI_HEAVY_S);
    munmap(stgl, uint64_t(n) * 4);
    munmap(grpl, uint64_t(n) * 4);
}

}  // namespace

int main() {
    classify(TRI_HEAVY_X + 1, 1, 2);
    classify(5000, 5000, 9);
    classify(1u << 26, 1u << 27, 1ull << 31);
    classify(1u << 27, 1u << 27, 1ull << 32);
    // beyond 2^27 tuples of S the ranges grow instead of their number, so that the items of all groups fit their word
    classify(1u << 27, 0xFFFFFFF0u, 1ull << 32);
    classify(0xFFFFFFF0u, 0xFFFFFFF0u, 1ull << 37);
    if (!fails) last_item();               // (with a 32-bit counter the queue would start again)
    std::printf("[heavy] %s\n", fails ? "FAILED" : "all checks passed");
    return fails ? 1 : 0;
}
