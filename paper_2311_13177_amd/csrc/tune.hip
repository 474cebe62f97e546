// Tile-shape autotuner of libvp: times steps with the compiled projection and gather tile shapes
// that fit a plan on the device and records the fastest per plan sizes. The shape only
// changes how the work is cut into work items (every shape gives the same bits), so the
// choice is purely a matter of speed.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <map>
#include <memory>
#include <mutex>
#include <tuple>
#include <vector>

#include "plan.h"
#include "runtime.h"

namespace vp {
namespace {

// What decides the fastest shape: sizes, the staged halo, the parts feeding a knot and
// the epilogue (Adam or GD). Plans with equal keys share a tuned shape.
struct TuneKey {
    int device, n, S, T, B, nparts, max_parts, hx, hy, optimizer;
    bool operator<(const TuneKey& o) const {
        return std::tie(device, n, S, T, B, nparts, max_parts, hx, hy, optimizer) <
               std::tie(o.device, o.n, o.S, o.T, o.B, o.nparts, o.max_parts, o.hx, o.hy, o.optimizer);
    }
};

std::mutex g_mu;
std::map<TuneKey, Tiles> g_tuned;

TuneKey key_of(const vp_plan* p, int device, int optimizer) {
    int hx = 0, hy = 0;
    for (const KnotInfo& k : p->knots) {
        hx = std::max(hx, k.ox_max - k.ox_min);
        hy = std::max(hy, k.oy_max - k.oy_min);
    }
    return TuneKey{device, p->n, p->S, p->T, p->B, p->nparts, p->max_knot_parts, hx, hy, optimizer};
}

int pow2_at_least(int v) {
    int r = 1;
    while (r < v) r <<= 1;
    return r;
}

// Every candidate is timed as whole steps, kRoundSteps at a time in kRounds rounds over all of them
// (the later ones over those near the fastest), by its least time. (Timed by itself, back to back, a kernel reads what its last launch has left in
// the Infinity Cache, which a step has streamed through, and shapes change places: 192^2 x 32 bins x 16
// knots in twelve rows takes 44 us in a step with eight waves, 49 with four, and its gather 192 us as
// 4 x 4 with eight, 197 as 2 x 8 with four; back to back either won. One pass alone times the first
// candidates while the clocks still rise.)
constexpr int kRounds = 3, kRoundSteps = 2;

}  // namespace

bool tuned_tiles(const vp_plan* p, int device, int optimizer, Tiles* out) {
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_tuned.find(key_of(p, device, optimizer));
    if (it == g_tuned.end()) return false;
    *out = it->second;
    return true;
}

vp_status tiles_for(const vp_plan* p, const vp_options* o, Tiles* out, bool* own) {
    if (own) *own = false;
    const vp_tiles& t = o->tiles;
    if (t.proj_rows || t.proj_parts || t.gath_rows || t.gath_bins || t.upd_bins || t.gath_waves || t.proj_waves ||
        t.gath_resident) {
        *out = Tiles{t.proj_rows, t.proj_parts, t.gath_rows, t.gath_bins, t.upd_bins,
                     t.gath_waves ? t.gath_waves : 4, t.proj_waves ? t.proj_waves : 4, t.gath_resident};
        return VP_OK;
    }
    if (tuned_tiles(p, o->device, o->optimizer, out)) return VP_OK;
    if (o->autotune) return tune_plan(p, o, out);
    if (own) *own = true;
    *out = p->base_tiles;
    return VP_OK;
}

vp_status tune_plan(const vp_plan* p, const vp_options* o, Tiles* out) {
    vp_status st = check_options(p, o);
    if (st != VP_OK) return st;
    hipError_t e = hipSetDevice(o->device);
    if (e != hipSuccess) return hip_status(e, "hipSetDevice");
    // scratch reconstruction state on the plan's built-in shape, zero measurements
    std::vector<vp_c64> zeros;
    try {
        zeros.assign(p->blade_px(), vp_c64{0.f, 0.f});
    } catch (const std::bad_alloc&) {
        return fail(VP_ERR_NOMEM, "autotune: out of host memory");
    }
    vp_options so = *o;
    so.tiles = vp_tiles{p->base_tiles.proj_rows, p->base_tiles.proj_gw, p->base_tiles.gath_rows,
                        p->base_tiles.gath_sc, 0, p->base_tiles.gath_w, p->base_tiles.proj_w,
                        p->base_tiles.gath_res};
    so.autotune = 0;
    vp_session* raw = nullptr;
    st = session_alloc(p, &so, zeros.data(), nullptr, nullptr, &raw);
    if (st != VP_OK) return st;
    std::unique_ptr<vp_session> s(raw);
    DeviceTables* tabs = s->tabs;

    if ((st = session_ensure_grad(s.get())) != VP_OK) return st;
    struct Events {
        hipEvent_t e0 = nullptr, e1 = nullptr;
        ~Events() {
            if (e0) (void)hipEventDestroy(e0);
            if (e1) (void)hipEventDestroy(e1);
        }
    } ev;
    e = hipEventCreate(&ev.e0);
    if (e == hipSuccess) e = hipEventCreate(&ev.e1);
    if (e != hipSuccess) return hip_status(e, "autotune events");

    // A candidate: a shape that fits the plan, its step, and the least time seen (ms).
    struct Candidate {
        Tiles t;
        StageLists lists;
        KArgs a{};
        float ms = FLT_MAX;
    };
    std::vector<Candidate> cand;
    auto offer = [&](const Tiles& t) -> vp_status {
        const Layout* L = nullptr;
        const DeviceLayout* dl = nullptr;
        if (plan_layout(p, t, &L) != VP_OK) {
            clear_error();
            return VP_OK;
        }
        const vp_status ls = device_layout(p, tabs, L, &dl);
        if (ls != VP_OK) return ls;
        Candidate c;
        c.t = t;
        c.lists = plan_lists(p, tabs, L, dl);
        c.lists.epi = s->lists.epi;
        c.lists.stream = s->lists.stream;
        c.a.one = s->desc;
        c.a.one.groups = dl->groups;
        try {
            cand.push_back(std::move(c));
        } catch (const std::bad_alloc&) {
            return fail(VP_ERR_NOMEM, "autotune: out of host memory");
        }
        return VP_OK;
    };
    // (a step of a blade-by-blade schedule has one blade's work: as many steps as blades, then)
    const int steps = o->schedule == VP_SCHED_ALL_BLADES ? kRoundSteps : std::min(p->B, 16);
    auto time_all = [&]() -> hipError_t {
        float least = FLT_MAX;
        for (int round = 0; round < kRounds; ++round)
            for (Candidate& c : cand) {
                if (round > 0 && c.ms > 1.1f * least) continue;  // out of reach
                float ms = 0.f;
                hipError_t te = hipEventRecord(ev.e0, s->stream);
                for (int i = 0; i < steps && te == hipSuccess; ++i) launch_step(c.a, c.lists, s->stream, &te);
                if (te == hipSuccess) te = hipEventRecord(ev.e1, s->stream);
                if (te == hipSuccess) te = hipEventSynchronize(ev.e1);
                if (te == hipSuccess) te = hipEventElapsedTime(&ms, ev.e0, ev.e1);
                if (te != hipSuccess) return te;
                c.ms = std::min(c.ms, ms);
                least = std::min(least, c.ms);
            }
        return hipSuccess;
    };
    // Times the candidates and leaves the fastest one's shape and time.
    auto choose = [&](Tiles* t, float* ms) -> vp_status {
        if ((e = time_all()) != hipSuccess) return hip_status(e, "autotune timing");
        for (const Candidate& c : cand)
            if (c.ms < *ms) {
                *ms = c.ms;
                *t = c.t;
            }
        cand.clear();
        return VP_OK;
    };

    // projection: every compiled (rows, parts per wave) with four and with eight waves per
    // item that keeps every wave busy (eight only where a knot has more than four parts)
    Tiles best = p->base_tiles;
    best.upd_sc = 0;
    float best_ms = FLT_MAX;
    for (int waves = 4; waves <= 8; waves += 4) {
        if (waves == 8 && p->max_knot_parts <= 4) break;
        const int gw_cap = std::min(8, pow2_at_least((std::max(1, p->max_knot_parts) + waves - 1) / waves));
        for (int rows : {1, 2, 4, 8, 12}) {
            for (int gw = 1; gw <= gw_cap; gw *= 2) {
                if (!proj_tiles_ok(rows, gw)) continue;
                Tiles t = p->base_tiles;
                t.proj_rows = rows;
                t.proj_gw = gw;
                t.proj_w = waves;
                if ((st = offer(t)) != VP_OK) return st;
            }
        }
    }
    if ((st = choose(&best, &best_ms)) != VP_OK) return st;
    // gather: every compiled (rows, bins per wave) with four and with eight waves per item
    // that keeps every wave busy, with the update fused (also with every part of a knot resident, where
    // the layout allows it), and storing the data gradient for a separate update pass; then every
    // update-pass shape
    auto offer_gathers = [&](bool resident, int upd_sc) -> vp_status {
        for (int waves = 4; waves <= 8; waves += 4) {
            // bins per wave up to the first power of two that covers S with every wave
            const int sc_cap = std::min(8, pow2_at_least((p->S + waves - 1) / waves));
            for (int rows = 2; rows <= 4; rows *= 2) {
                for (int sc = 1; sc <= sc_cap; sc *= 2) {
                    if (!gath_tiles_ok(rows, sc, resident)) continue;
                    Tiles t = best;
                    t.gath_rows = rows;
                    t.gath_sc = sc;
                    t.gath_w = waves;
                    t.upd_sc = upd_sc;
                    t.gath_res = resident;
                    const vp_status os = offer(t);
                    if (os != VP_OK) return os;
                }
            }
        }
        return VP_OK;
    };
    Tiles fused = best, split = best;
    float fused_ms = FLT_MAX, split_ms = FLT_MAX;
    for (bool resident : {false, true})
        if ((st = offer_gathers(resident, 0)) != VP_OK) return st;
    if ((st = choose(&fused, &fused_ms)) != VP_OK) return st;
    if ((st = offer_gathers(false, 4)) != VP_OK) return st;
    if ((st = choose(&split, &split_ms)) != VP_OK) return st;
    for (int usc : {2, 8}) {
        Tiles t = split;
        t.upd_sc = usc;
        if ((st = offer(t)) != VP_OK) return st;
    }
    if ((st = choose(&split, &split_ms)) != VP_OK) return st;
    best = split_ms < fused_ms ? split : fused;
    if ((e = hipStreamSynchronize(s->stream)) != hipSuccess) return hip_status(e, "autotune");
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_tuned[key_of(p, o->device, o->optimizer)] = best;
    }
    *out = best;
    return VP_OK;
}

}  // namespace vp

using namespace vp;

static vp_tiles to_abi(const Tiles& t) {
    return vp_tiles{t.proj_rows, t.proj_gw, t.gath_rows, t.gath_sc, t.upd_sc, t.gath_w, t.proj_w, t.gath_res};
}

extern "C" vp_status vp_plan_tune(const vp_plan* p, const vp_options* o, vp_tiles* out) {
    clear_error();
    if (!p || !o || !out) return fail(VP_ERR_ARG, "vp_plan_tune: NULL argument");
    Tiles t;
    const vp_status st = tune_plan(p, o, &t);
    if (st == VP_OK) *out = to_abi(t);
    return st;
}

extern "C" vp_status vp_plan_tiles(const vp_plan* p, const vp_options* o, vp_tiles* out) {
    clear_error();
    if (!p || !o || !out) return fail(VP_ERR_ARG, "vp_plan_tiles: NULL argument");
    vp_status st = check_options(p, o);
    if (st != VP_OK) return st;
    Tiles t;
    st = tiles_for(p, o, &t);
    if (st != VP_OK) return st;
    const Layout* L = nullptr;
    st = plan_layout(p, t, &L);
    if (st == VP_OK) *out = to_abi(t);
    return st;
}
