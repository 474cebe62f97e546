// Enumerates tile shapes over geometries read from stdin and prints every accepted layout whose
// largest projection region the launch would refuse or stage past its LDS plane.
//
// stdin: geometries as "n S T B  shift[S] angle[B] time[B]" (lines: one per blade).
#include <algorithm>
#include <cstdio>
#include <vector>

#include "plan.h"

using namespace vp;

namespace {

int extent(int rows, const ProjGroup& g, bool even) {
    const int x0 = even ? g.ox_min & ~1 : g.ox_min, x1 = even ? g.ox_max | 1 : g.ox_max;
    return (rows + g.oy_max - g.oy_min + 1) * (kTileW + x1 - x0 + 1);
}

}  // namespace

int main() {
    int n, S, T, B, accepted = 0, bad = 0, at_limit = 0;
    while (scanf("%d %d %d %d", &n, &S, &T, &B) == 4) {
        std::vector<double> shift(S), angle(B), time(B);
        for (auto* v : {&shift, &angle, &time})
            for (double& x : *v)
                if (scanf("%lf", &x) != 1) return 2;
        std::vector<int> lines(B, 1);
        vp_geometry g{};
        g.n = n; g.n_spec = S; g.n_time = T; g.n_blades = B;
        g.angle_rad = angle.data(); g.lines = lines.data(); g.spec_shift_px = shift.data();
        g.blade_time = T > 1 ? time.data() : nullptr;
        vp_plan* p = nullptr;
        if (vp_plan_create(&g, &p) != VP_OK) { printf("plan refused: %s\n", vp_last_error()); return 2; }
        for (int rows : {1, 2, 4, 8, 12})
            for (int gw : {1, 2, 4, 8})
                for (int waves : {4, 8}) {
                    Tiles t;
                    t.proj_rows = rows; t.proj_gw = gw; t.proj_w = waves;
                    const Layout* L = nullptr;
                    if (plan_layout(p, t, &L) != VP_OK) continue;
                    ++accepted;
                    int exact = 1, even = 1;
                    for (const ProjGroup& gr : L->groups) {
                        exact = std::max(exact, extent(rows, gr, false));
                        even = std::max(even, extent(rows, gr, true));
                    }
                    const int limit = kStageMax * kThreads;
                    at_limit += exact <= limit && even > limit;
                    // 16-byte units (even n, up to half the limit) stage the even region
                    const bool wide = n % 2 == 0 && L->re_proj <= limit / 2;
                    if (L->re_proj < 1 || L->re_proj > limit || L->re_proj < (wide ? even : exact)) {
                        ++bad;
                        printf("n %d rows %d gw %d waves %d: region %d (exact %d, even %d)\n", n, rows, gw, waves,
                               L->re_proj, exact, even);
                    }
                }
        vp_plan_destroy(p);
    }
    printf("accepted %d at_limit %d bad %d\n", accepted, at_limit, bad);
    return bad ? 1 : 0;
}
