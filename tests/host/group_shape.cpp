// The kernels of a batch's step and of a slice's alone, with stand-in runtime functions: a shape
// that was asked for is the one that runs, also where it is the one the plan would take by itself.
#include <cstdio>
#include <vector>

#include "fake_hip.h"
#include "vp.h"

int main() {
    const int n = 64, S = 16, B = 5, K = 24;
    std::vector<double> angle(B), shift(S);
    std::vector<int32_t> lines(B, 8);
    for (int b = 0; b < B; ++b) angle[b] = 3.14159265358979 * b / B;
    for (int s = 0; s < S; ++s) shift[s] = 0.1 * s;
    vp_geometry g{};
    g.n = n; g.n_spec = S; g.n_time = 1; g.n_blades = B;
    g.angle_rad = angle.data(); g.lines = lines.data(); g.spec_shift_px = shift.data();
    vp_plan* p = nullptr;
    if (vp_plan_create(&g, &p) != VP_OK) return 2;
    std::vector<vp_c64> y((size_t)B * n * n, vp_c64{0.f, 0.f});
    vp_options own{};
    if (vp_options_default(&own) != VP_OK) return 2;
    own.n_steps = 4;
    vp_tiles t{};
    if (vp_plan_tiles(p, &own, &t) != VP_OK) return 2;
    vp_options asked = own;
    asked.tiles = t;

    // (the projection is a step's first kernel, the gather its last)
    auto solo = [&](const vp_options& o) {
        vp_session* s = nullptr;
        if (vp_session_create(p, &o, y.data(), nullptr, &s) != VP_OK) { printf("%s\n", vp_last_error()); exit(2); }
        g_launches.clear();
        if (vp_session_step(s, 1, 0) != VP_OK) exit(2);
        const std::vector<Launch> l = g_launches;
        vp_session_destroy(s);
        return l;
    };
    auto batch = [&](const vp_options& o) {
        std::vector<const vp_plan*> ps(K, p);
        std::vector<const vp_options*> os(K, &o);
        std::vector<const vp_c64*> ys(K, y.data());
        vp_batch* b = nullptr;
        if (vp_batch_create(K, ps.data(), os.data(), ys.data(), &b) != VP_OK) { printf("%s\n", vp_last_error()); exit(2); }
        g_launches.clear();
        if (vp_batch_step(b, 1, 0) != VP_OK) exit(2);
        const std::vector<Launch> l = g_launches;
        vp_batch_destroy(b);
        return l;
    };
    const auto one = solo(asked), all = batch(asked), mine = batch(own);
    const bool kept = all.front().kernel == one.front().kernel && all.back().kernel == one.back().kernel &&
                      all.front().grid.x == K * one.front().grid.x;
    const bool follows = mine.front().kernel != one.front().kernel && mine.back().kernel != one.back().kernel;
    printf("asked shape %s, own shape %s\n", kept ? "kept" : "replaced", follows ? "follows the group" : "does not");
    vp_plan_destroy(p);
    return kept && follows ? 0 : 1;
}
