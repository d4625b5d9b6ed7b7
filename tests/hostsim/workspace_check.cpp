// Host-build check of planned workspaces (test infrastructure only): a small
// linear join's plan asks for no room for the hashed tables' narrow forms,
// whose least size (32 bytes for each of 2^19 slots) is several times all the
// rest, and the autotuner still tries every bucket count in that workspace.
#include <cstdio>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#include "mj.h"

static int fails = 0;
static void expect(bool ok, const char* what, double got) {
    std::printf("[workspace] %-66s %s (%.2f)\n", what, ok ? "ok" : "FAILED", got);
    if (!ok) ++fails;
}

int main() {
    constexpr uint64_t narrow = 32ull << 19;
    for (uint64_t n : {5000ull, 20000ull})
        for (int sparse = 0; sparse < 2; ++sparse) {
            mj_ctx* ctx = nullptr;                    // (of its own: it keeps tuned plans by size class)
            if (mj_ctx_create(0, &ctx) != MJ_OK) return 2;
            std::mt19937 g((uint32_t)n);
            std::vector<uint32_t> R(2 * n), S(2 * n), T(2 * n);
            for (uint64_t i = 0; i < 2 * n; ++i) {
                R[i] = g() % 900; S[i] = g() % 900; T[i] = g() % 900;
                if (sparse) { if (i & 1) R[i] *= 2654435761u; S[i] *= 2654435761u; T[i] *= 2654435761u; }
            }
            mj_rel r{R.data(), R.data() + 1, n, 2}, s{S.data(), S.data() + 1, n, 2}, t{T.data(), T.data() + 1, n, 2};
            std::vector<unsigned char> pws(mj_plan_workspace(MJ_LINEAR, n, n, n));
            mj_plan_t p;
            std::memset(&p, 0, sizeof p);
            expect(mj_plan(ctx, MJ_LINEAR, &r, &s, &t, 900, MJ_PLANNER_ANALYTIC, &p, pws.data(), pws.size(), nullptr) ==
                       MJ_OK && ((p.flags & MJ_PLAN_DENSE_KEYS) != 0) == !sparse, "plan", (double)n);
            expect(p.workspace_bytes - 8 * p.join2_size < narrow,
                   "workspace without the intermediate, MB: below the narrow forms'",
                   (p.workspace_bytes - 8 * p.join2_size) / 1e6);
            std::vector<unsigned char> ws(p.workspace_bytes);
            std::vector<uint64_t> want(900), out(900);
            expect(mj_linear3_count(ctx, &r, &s, &t, 900, want.data(), &p, ws.data(), ws.size(), nullptr) == MJ_OK,
                   "count in the planned workspace", 0);
            mj_ctx_profile(ctx, 1);
            std::vector<char> names(64 * 32);
            std::vector<double> ms(64);
            std::vector<int64_t> launches(64);
            mj_ctx_profile_read(ctx, 64, names.data(), ms.data(), launches.data());
            double t_ms = 0;
            mj_plan_t q = p;
            expect(mj_autotune(ctx, MJ_LINEAR, &r, &s, &t, 900, out.data(), &q, ws.data(), ws.size(), &t_ms, nullptr) ==
                       MJ_OK && out == want, "autotuner in the planned workspace: the same counts", 0);
            const int k = mj_ctx_profile_read(ctx, 64, names.data(), ms.data(), launches.data());
            mj_ctx_profile(ctx, 0);
            int64_t counts = 0;
            for (int i = 0; i < k; ++i) if (std::string(&names[32 * i]) == "k_count") counts = launches[i];
            // nine pairs of bucket counts, a warm-up and two timed runs each
            expect(counts >= 27, "runs of the hashed join (three of each candidate)", (double)counts);
            mj_ctx_destroy(ctx);
        }
    std::printf("[workspace] %s\n", fails ? "FAILED" : "all checks passed");
    return fails ? 1 : 0;
}
