// Host-side plan of libvp: validated geometry, FP64-derived tables and launch lists.
#pragma once

#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "vp.h"
#include "vp_internal.h"

namespace vp {

// Sets the thread-local error message and returns `code`.
vp_status fail(vp_status code, const char* fmt, ...);
void clear_error();

// Tile shape of the projection and gather work items (see vp_internal.h). Results never
// depend on it: only the work decomposition changes.
struct Tiles {
    int proj_rows = 2, proj_gw = 1, gath_rows = 2, gath_sc = 1;
    int upd_sc = 0;  // 0: update fused into the gather; else bins per wave of the update pass
    int gath_w = 4;  // waves per gather item
    int proj_w = 4;  // waves per projection item
    int gath_res = 0;  // 1: the resident-parts gather (every part of a knot staged at once)
    int key() const {
        return proj_rows | proj_gw << 4 | gath_rows << 8 | gath_sc << 12 | upd_sc << 16 | gath_w << 20 | proj_w << 24 |
               gath_res << 28;
    }
    bool operator==(const Tiles& o) const { return key() == o.key(); }
};

// Projection groups and work lists of one tile shape.
struct Layout {
    Tiles tiles;
    std::vector<ProjGroup> groups;
    std::vector<Task> t_proj, t_gath, t_upd;
    int re_proj = 0, re_gath = 0;  // largest staged region (elements) of an item
    size_t lds_res = 0;            // resident-parts gather: LDS bytes of the largest knot
};

// A layout's tables on one device.
struct DeviceLayout {
    void* base = nullptr;
    ProjGroup* groups = nullptr;
    Task* t_proj = nullptr;
    Task* t_gath = nullptr;
    Task* t_upd = nullptr;
    ~DeviceLayout();
};

// Workspaces that the operator calls of a plan keep on one device, so that a call pays neither an
// allocation nor a free (24 us of host time a pair; a 64^2 forward's three launches take 14 us).
// A slot belongs to one stream and to one call at a time; a call takes the smallest that
// fits (blade-aligned calls hold two, of different sizes). The call that takes it again first waits,
// on its stream, for the event of the call before, so a stream made at a destroyed one's
// address is safe too. Where a stream has none and no slot is empty, it takes one over that is idle
// and whose last call is done on the device (streams come and go; at once one that fits, else
// replaced by one that does). A call gets stream-ordered memory of its own instead while its stream
// is captured (a graph's workspace may not be shared with later calls), on the per-thread default
// stream, above kKeepBytes (there the kernels take 300 us and more and the host runs ahead), and
// where all kSlots are at work. The slots are freed with the plan.
struct WorkspaceSlots {
    static constexpr int kSlots = 4;
    static constexpr size_t kKeepBytes = (size_t)64 << 20;
    struct Slot {
        void* ptr = nullptr;
        size_t bytes = 0;
        hipStream_t stream = nullptr;
        hipEvent_t done = nullptr;
        bool busy = false;
        uint64_t used = 0;  // the call that took it last
    };
    std::mutex mu;
    Slot slot[kSlots];
    uint64_t calls = 0;
    int claim(size_t bytes, hipStream_t s);
    ~WorkspaceSlots();
};
// One call's workspace: a slot, or stream-ordered memory.
struct Workspace {
    WorkspaceSlots* from = nullptr;
    int slot = -1;
    void* ptr = nullptr;
    hipStream_t s = nullptr;
    hipError_t take(WorkspaceSlots* slots, size_t bytes, hipStream_t stream);
    ~Workspace();
};

// Per-device copies of a plan's constant tables and work lists (one allocation for the tables here,
// one for those of blade-aligned sampling).
struct DeviceTables {
    int device = -1;
    void* base = nullptr;
    void* nu_base = nullptr;
    uint8_t* mask = nullptr;
    ShearEntry* shear = nullptr;
    BladeDev* blade = nullptr;
    int* knot_ptr = nullptr;
    KnotEntry* knot_ent = nullptr;
    ShearEntry* knot_tap = nullptr;
    KnotInfo* knots = nullptr;
    float2* tw = nullptr;
    Task* t_rows = nullptr;
    Task* t_cols = nullptr;
    Task* t_vox = nullptr;
    Task* t_render = nullptr;
    std::map<int, std::unique_ptr<DeviceLayout>> layouts;  // by Tiles::key()
    // blade-aligned sampling tables (uploaded on first use)
    int* nu_lines = nullptr;
    double2* nu_cs = nullptr;
    float2* nu_ph = nullptr;
    float* nu_dea = nullptr;
    float* nu_kb = nullptr;
    Task* nu_rows = nullptr;
    WorkspaceSlots work;
    ~DeviceTables();
};

// Host tables of blade-aligned sampling (see the blade-sampling kernels).
struct NuHost {
    int lmax = 0;
    float kmax = 0.f;
    std::vector<int> lines;
    std::vector<double2> cs;         // [B]
    std::vector<float2> ph;          // [B][lmax][n]
    std::vector<float> dea, kb;      // [n], [kNuTable + 1]
    std::vector<Task> rows;          // row-pass tasks of the oversampled plan that touch the image's rows
};

}  // namespace vp

struct vp_plan {
    int n = 0, S = 0, T = 0, B = 0;
    std::vector<double> angle, tau, shift;
    std::vector<int> lines;
    std::vector<uint8_t> mask;           // [B][n][n]
    std::vector<vp::ShearEntry> shear;   // [B][S]
    std::vector<float> fx, fy;           // [B][S] fractional parts, for inspection
    std::vector<vp::BladeDev> blade;     // [B]
    std::vector<float> alpha;            // [B]
    std::vector<int> knot_ptr;           // [T+1]
    std::vector<vp::KnotEntry> knot_ent;
    std::vector<vp::ShearEntry> knot_tap;  // [entries][S]: the blade's taps times the entry weight
    std::vector<vp::KnotInfo> knots;    // [T]
    int max_knot_parts = 0;              // most blade parts feeding one knot
    std::vector<float2> tw;              // [n]
    int nstage = 0;
    int radix[vp::kMaxStages] = {0};
    int nparts = 1;
    int n_col_items = 0;
    // Work lists of the tile-independent stages (slice index 0; batches rebase it).
    std::vector<vp::Task> t_rows, t_cols, t_vox, t_render;
    // Dynamic LDS bytes per kernel.
    size_t lds_rows = 0, lds_cols = 0;
    // The layout of the default tile shape, built and checked at creation.
    vp::Tiles base_tiles;

    mutable std::mutex mu;
    mutable std::map<int, std::unique_ptr<vp::Layout>> layouts;  // host layouts by Tiles::key()
    mutable std::map<int, std::unique_ptr<vp::DeviceTables>> dev;
    // The same geometry with a knot per blade (built on first use; K-Planes fits).
    mutable std::mutex mu_derived;
    mutable std::unique_ptr<vp_plan> per_blade;
    // Blade-aligned sampling: its host tables and the plan of the oversampled grid
    // (2n x 2n, the same blades; its DFT passes only), built on first use.
    mutable std::unique_ptr<vp::NuHost> nu_host;
    mutable std::unique_ptr<vp_plan> over;

    uint64_t voxels() const { return (uint64_t)T * S * n * n; }
    uint64_t blade_px() const { return (uint64_t)B * n * n; }
};

namespace vp {

// The plan's geometry with one knot per blade (knot b holds blade b with weight 1, one
// work part per blade), built on first use and kept with the plan.
vp_status plan_per_blade(const vp_plan* plan, const vp_plan** out);
// Blade-aligned sampling: host tables and the oversampled grid's plan (VP_ERR_UNSUPPORTED
// if 2n exceeds the largest transform length).
vp_status plan_nu(const vp_plan* plan, const NuHost** host, const vp_plan** over);
// The tables of plan_nu on the device of `t`, uploaded on first use.
vp_status nu_tables(const vp_plan* plan, const NuHost* host, DeviceTables* t);

// Device tables of `plan` on the current device, uploading them on first use.
vp_status plan_tables(const vp_plan* plan, DeviceTables** out);

// Host layout of `plan` for tile shape `t` (built on first use and kept with the plan).
// VP_ERR_UNSUPPORTED if the shape is not compiled or a staged region would not fit.
vp_status plan_layout(const vp_plan* plan, const Tiles& t, const Layout** out);
// A layout's tables on the device of `tabs`, uploaded on first use.
vp_status device_layout(const vp_plan* plan, DeviceTables* tabs, const Layout* L, const DeviceLayout** out);
// Rows, parts per wave and waves of the projection items for one launch over these plans.
void proj_shape_for(const std::vector<const vp_plan*>& plans, Tiles* t);
// Rows by bins of a wave of the gather: the resident one keeps a bin's sums at a time; the phased
// one all of them, beside the update's registers where it is fused (384^2 x 64 bins x 24 blades: 4 x 4
// 227 us, 4 x 2 207 us, x 8 knots 1062 and 1007 us) and alone where it stores (384^2 x 64 x 8 knots with
// the update pass: 4 x 4 1153 us, 4 x 2 1209 us).
constexpr int kResidentSums = 32, kPhasedStore = 16, kPhasedStep = 8;
// The plan's own shape where the gather only stores (operators, K-Planes).
Tiles store_tiles(const vp_plan* plan);
// A plan's own shape t for one step's launches over all of these plans (S: bins of the largest).
Tiles group_shape(Tiles t, const std::vector<const vp_plan*>& plans, int S);
// Tile shape chosen without measuring, from the plan's sizes, with the resident or the phased gather.
Tiles heuristic_tiles(const vp_plan* plan, bool resident);

// Fills the plan-constant part of a slice descriptor from device tables and a layout.
void fill_desc(const vp_plan* plan, const DeviceTables* t, const Layout* L, const DeviceLayout* dl, SliceDesc* d);

// Loss partial slots (floats) per reconstruction.
inline uint64_t loss_slots(const vp_plan* p) { return (uint64_t)p->B * p->n_col_items; }

}  // namespace vp
