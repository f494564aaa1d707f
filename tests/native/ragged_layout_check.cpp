// The ragged launch's role order over batches around its lag (the plain call's):
// every role of every element once, and each after what it waits on.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "plan.hpp"

using namespace sv;

static void fail(const char* what, int B, int gamma, int V) {
    printf("%s at B=%d gamma=%d V=%d\n", what, B, gamma, V);
    exit(1);
}

static void check(int B, int gamma, int V, sv_dtype_t dt) {
    Plan p{};
    if (!make_plan(B, gamma, V, dt, &p)) fail("no plan", B, gamma, V);
    const Layout y = single_pass_layout(B, gamma, V, dt, true, p);
    const long long unit = 2LL * gamma * V * bytes_per_logit(dt);
    if (y.lagM != std::min<long long>(B, ceil_div(kLagStreamBytes, unit)) || y.lagM < 1 || y.lagM > B) fail("lag", B, gamma, V);
    const int S = 2 * gamma * p.nchunk1;
    std::vector<long long> last_stats(B, -1), decider(B, -1), draw(B, -1), bonus(B, -1);
    std::vector<int> stats((size_t)B * S), mass((size_t)B * p.nchunk2), rowg((size_t)B * p.nchunkg);
    std::vector<long long> first_mass(B, -1), last_mass(B, -1), last_g(B, -1);
    const long long n = (long long)y.end2 + B;
    for (long long id = 0; id < n; ++id) {
        const Role r = role_at(y, p.nchunk1, p.nchunkg, (unsigned int)id);
        if (r.b < 0 || r.b >= B) fail("element", B, gamma, V);
        switch (r.kind) {
            case kRoleStats: ++stats.at((size_t)r.b * S + (size_t)r.slot * p.nchunk1 + r.k); last_stats[r.b] = id; break;
            case kRoleRowG: ++rowg.at((size_t)r.b * p.nchunkg + r.k); last_g[r.b] = id; break;
            case kRoleMass:
                ++mass.at((size_t)r.b * p.nchunk2 + r.k);
                if (first_mass[r.b] < 0) first_mass[r.b] = id;
                last_mass[r.b] = id;
                break;
            case kRoleDecider: if (decider[r.b] >= 0) fail("decider", B, gamma, V); decider[r.b] = id; break;
            case kRoleDraw: if (draw[r.b] >= 0) fail("draw", B, gamma, V); draw[r.b] = id; break;
            case kRoleBonus: if (bonus[r.b] >= 0) fail("bonus", B, gamma, V); bonus[r.b] = id; break;
            default: fail("role", B, gamma, V);
        }
    }
    for (const auto* v : {&stats, &mass, &rowg})
        for (int c : *v)
            if (c != 1) fail("a role not once", B, gamma, V);
    for (int b = 0; b < B; ++b)
        if (!(last_stats[b] < decider[b] && decider[b] < first_mass[b] && last_mass[b] < draw[b] &&
              decider[b] < bonus[b] && last_g[b] < bonus[b]))
            fail("order", B, gamma, V);
}

int main() {
    const struct { int gamma, V; sv_dtype_t dt; } shapes[] = {
        {1, 51865, SV_F32}, {2, 100000, SV_BF16}, {8, 128256, SV_BF16}, {20, 65001, SV_F16}, {7, 131073, SV_F32}, {3, 9, SV_F32}};
    for (const auto& s : shapes) {
        const long long lag = ceil_div(kLagStreamBytes, 2LL * s.gamma * s.V * bytes_per_logit(s.dt));
        for (long long B : {1LL, 2LL, 9LL, lag - 1, lag, lag + 1, 2 * lag})
            if (B >= 1 && B <= 700) check((int)B, s.gamma, s.V, s.dt);
    }
    printf("all checks passed\n");
}
