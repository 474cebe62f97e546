// The kernels of a batch's step and of a slice's alone, with stand-in runtime functions: a shape
// that was asked for is the one that runs, also where it is the one the plan would take by itself.
#include <cstdio>
#include <vector>

#include "fake_hip.h"
#include "vp.h"

struct Scan {
    vp_plan* p = nullptr;
    std::vector<vp_c64> y;
    vp_options own{};
    Scan(int n, int S, int B, double step);
    ~Scan() { vp_plan_destroy(p); }
    std::vector<Launch> solo(const vp_options& o) const;
    std::vector<Launch> batch(const vp_options& o, int K) const;
};

Scan::Scan(int n, int S, int B, double step) {
    std::vector<double> angle(B), shift(S);
    std::vector<int32_t> lines(B, 8);
    for (int b = 0; b < B; ++b) angle[b] = 3.14159265358979 * b / B;
    for (int s = 0; s < S; ++s) shift[s] = step * s;
    vp_geometry g{};
    g.n = n; g.n_spec = S; g.n_time = 1; g.n_blades = B;
    g.angle_rad = angle.data(); g.lines = lines.data(); g.spec_shift_px = shift.data();
    if (vp_plan_create(&g, &p) != VP_OK || vp_options_default(&own) != VP_OK) exit(2);
    own.n_steps = 4;
    y.assign((size_t)B * n * n, vp_c64{0.f, 0.f});
}

// (the projection is a step's first kernel, the gather its last)
std::vector<Launch> Scan::solo(const vp_options& o) const {
    vp_session* s = nullptr;
    if (vp_session_create(p, &o, y.data(), nullptr, &s) != VP_OK) { printf("%s\n", vp_last_error()); exit(2); }
    g_launches.clear();
    if (vp_session_step(s, 1, 0) != VP_OK) exit(2);
    const std::vector<Launch> l = g_launches;
    vp_session_destroy(s);
    return l;
}

std::vector<Launch> Scan::batch(const vp_options& o, int K) const {
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
}

int main() {
    const int K = 24;
    const Scan small(64, 16, 5, 0.1);
    vp_options asked = small.own;
    if (vp_plan_tiles(small.p, &small.own, &asked.tiles) != VP_OK) return 2;
    const auto one = small.solo(asked), all = small.batch(asked, K), mine = small.batch(small.own, K);
    const bool kept = all.front().kernel == one.front().kernel && all.back().kernel == one.back().kernel &&
                      all.front().grid.x == K * one.front().grid.x;
    const bool follows = mine.front().kernel != one.front().kernel && mine.back().kernel != one.back().kernel;

    const Scan wide(96, 16, 16, 0.25);
    vp_options phased = wide.own;
    phased.tiles = vp_tiles{4, 1, 4, 2, 0, 8, 8, 0};
    vp_tiles t{};
    if (vp_plan_tiles(wide.p, &wide.own, &t) != VP_OK) return 2;
    const bool large = t.gath_resident == 1 && t.gath_rows == 2 &&
                       wide.batch(wide.own, 6).back().kernel == wide.solo(phased).back().kernel;
    printf("asked shape %s, own shape %s, phased %s\n", kept ? "kept" : "replaced",
           follows ? "follows the group" : "does not", large ? "at its size" : "at another");
    return kept && follows && large ? 0 : 1;
}
