// The tuner's choice of projection and gather, with stand-in runtime functions and a cost per launch:
// a kernel that follows its like reads what that one left in the caches, and is then fastest with
// four waves; behind any other kernel, as in a step, it is fastest with eight.
#include <cstdio>
#include <set>

#include "fake_hip.h"
#include "vp.h"

static std::set<const void*> g_projections, g_gathers;

static float cost(size_t i) {
    const Launch& l = g_launches[i];
    for (const auto* like : {&g_projections, &g_gathers}) {
        if (!like->count(l.kernel)) continue;
        const bool warm = i > 0 && like->count(g_launches[i - 1].kernel);
        const bool eight = l.block.x == 512;
        return warm == eight ? 2.f : 1.f;
    }
    return 1.f;
}

int main() {
    const int n = 96, S = 8, B = 6;
    std::vector<double> angle(B), shift(S);
    std::vector<int32_t> lines(B, 8);
    for (int b = 0; b < B; ++b) angle[b] = 3.14159265358979 * b / B;
    for (int s = 0; s < S; ++s) shift[s] = 0.2 * s;
    vp_geometry g{};
    g.n = n; g.n_spec = S; g.n_time = 1; g.n_blades = B;
    g.angle_rad = angle.data(); g.lines = lines.data(); g.spec_shift_px = shift.data();
    vp_plan* p = nullptr;
    if (vp_plan_create(&g, &p) != VP_OK) return 2;
    vp_options o{};
    if (vp_options_default(&o) != VP_OK) return 2;
    o.n_steps = 4;
    // the kernels of every shape: an eager step's first is the projection, its last the gather
    std::vector<vp_c64> y((size_t)B * n * n, vp_c64{0.f, 0.f});
    auto step = [&](const vp_tiles& t) {
        vp_options a = o;
        a.tiles = t;
        vp_session* s = nullptr;
        if (vp_session_create(p, &a, y.data(), nullptr, &s) != VP_OK) return;
        g_launches.clear();
        if (vp_session_step(s, 1, 0) != VP_OK) exit(2);
        g_projections.insert(g_launches.front().kernel);
        g_gathers.insert(g_launches[g_launches.size() - (t.upd_bins ? 2 : 1)].kernel);
        vp_session_destroy(s);
    };
    for (int rows : {1, 2, 4, 8, 12})
        for (int k : {1, 2, 4, 8})
            for (int waves : {4, 8}) {
                step(vp_tiles{rows, k, 2, 1, 0, 4, waves, 0});
                for (int upd : {0, 2})
                    for (int res : {0, 1}) step(vp_tiles{2, 1, rows, k, upd, waves, 4, res});
            }
    g_launches.clear();
    g_cost = cost;
    vp_tiles t{};
    if (vp_plan_tune(p, &o, &t) != VP_OK) { printf("%s\n", vp_last_error()); return 2; }
    printf("%zu projections, %zu gathers, tuned to %d and %d waves\n", g_projections.size(), g_gathers.size(),
           t.proj_waves, t.gath_waves);
    vp_plan_destroy(p);
    return t.proj_waves == 8 && t.gath_waves == 8 ? 0 : 1;
}
