// Internal declarations shared by the runtime, batch and server translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "plan.h"

namespace vp {

// Kernel launchers (kernels.hip).
// re: largest staged region (elements) over the work items' slices.
// waves: 4 or 8 per work item (the layout's proj_w: its groups hold waves * gw parts)
// odd: whether any slice of the launch has an odd n
hipError_t launch_project(const KArgs& a, int rows, int gw, int waves, int re, bool odd, hipStream_t s);
// n: the length of every slice of the launch, or kFftMixed (lds: the largest over the slices).
hipError_t launch_rows(const KArgs& a, int dir, int n, size_t lds, hipStream_t s);
hipError_t launch_cols(const KArgs& a, int n, size_t lds, hipStream_t s);
// Every blade of one slice (a.one) through the passes of a.mode, one block each (n <= kBladeN).
hipError_t launch_blades(const KArgs& a, hipStream_t s);
// Whether a length has compile-time passes.
bool fft_compiled(int n);
// waves: 4 or 8 per work item (the layout's gath_w: its bin chunks hold waves * sc bins)
hipError_t launch_gather(const KArgs& a, int mode, int rows, int sc, int waves, int re, hipStream_t s);
// The resident-parts gather: lds bytes of the largest knot's parts (Layout::lds_res).
// re: largest staged region (elements) of the layout (re_gath).
hipError_t launch_gather_res(const KArgs& a, int mode, int rows, int sc, int waves, int re, size_t lds, hipStream_t s);
hipError_t launch_update(const KArgs& a, int sc, hipStream_t s);
hipError_t launch_tv_grad(const KArgs& a, hipStream_t s);
hipError_t launch_reg_value(const KArgs& a, hipStream_t s);
hipError_t launch_render(const KArgs& a, hipStream_t s);
hipError_t launch_baseline_avg(const uint8_t* mask, const float2* y, float2* out, int n, int window, int first,
                               int n_frames, hipStream_t s);
hipError_t launch_psnr(const float2* img, const float2* truth, long long npx, int n_images, double* terms,
                       hipStream_t s);

// The row and column passes of a launch over slices of several lengths: items [rows0, rows0 +
// n_rows) and [cols0, cols0 + n_cols) have length n (kFftMixed: several of the lengths up to 384
// with a compile-time plan; 0: any without one).
struct FftSegment {
    int n = 0, rows0 = 0, n_rows = 0, cols0 = 0, n_cols = 0;
    size_t lds_rows = 0, lds_cols = 0;
};

// Device work lists of one optimiser step and the dynamic LDS of each stage.
struct StageLists {
    const Task* proj = nullptr;
    const Task* rows = nullptr;
    const Task* cols = nullptr;
    const Task* gath = nullptr;
    const Task* vox = nullptr;
    const Task* render = nullptr;
    const Task* upd = nullptr;
    int n_slices = 1;  // slices whose step counters the step advances
    int n_proj = 0, n_rows = 0, n_cols = 0, n_gath = 0, n_vox = 0, n_render = 0, n_upd = 0;
    Tiles tiles;
    bool odd = false;  // whether any slice has an odd n
    int fft_n = 0;  // length of the slice (of a group's first)
    size_t lds_rows = 0, lds_cols = 0;
    std::vector<FftSegment> segs;  // a group's lengths (empty: one slice)
    int re_proj = 0, re_gath = 0;  // largest staged regions (elements)
    size_t lds_res = 0;            // resident-parts gather: LDS bytes of the largest knot
    int epi = EPI_GENERIC;         // optimiser epilogue every slice of the step can take
    int stream = 0;                // the step's state exceeds kStreamState (EPI_STREAM)
};

// Whether a launch's row and column passes are one (launch_blades): one slice of a small length.
inline bool blades_whole(const KArgs& a, const StageLists& L) {
    return !a.descs && L.segs.empty() && L.fft_n <= kBladeN;
}
// One slice's row and column passes: COL_STEP (work to work, the inverse rows left to the caller
// unless blades_whole), COL_FORWARD (work to a.out0) or COL_ADJOINT (a.in0 to work).
hipError_t launch_blur(KArgs a, const StageLists& L, int mode, hipStream_t s);

StageLists plan_lists(const vp_plan* p, const DeviceTables* t, const Layout* L, const DeviceLayout* dl);
// Whether a step over `voxels` voxels (summed over its slices) streams its state.
inline int stream_for(uint64_t voxels, int optimizer) {
    return voxels * sizeof(float2) * (optimizer == VP_OPT_ADAM ? 4u : 2u) > kStreamState ? 1 : 0;
}
// The gather of a step's layout (resident-parts or staged a few parts at a time).
hipError_t launch_gather_lists(const KArgs& a, int mode, const StageLists& L, hipStream_t s);
// Tile shape for a plan under options: explicit tiles from the options, else the tuned
// shape recorded for this plan's sizes on the device (tuning first when the options ask
// for it and none is recorded), else the plan's heuristic shape (*own: whether that one).
vp_status tiles_for(const vp_plan* p, const vp_options* o, Tiles* out, bool* own = nullptr);
// Tuned shape recorded for the plan's sizes on `device`, if any.
bool tuned_tiles(const vp_plan* p, int device, int optimizer, Tiles* out);
// Measures the candidate tile shapes on the current device and records the fastest.
vp_status tune_plan(const vp_plan* p, const vp_options* o, Tiles* out);
// Enqueues one optimiser step (project, row DFT, column pass, inverse row DFT,
// gather + update, the last also advancing the step counters) for the descriptors
// `base` refers to.
// With `ev` (kStages + 1 events) an event is recorded before each stage and after the last.
void launch_step(const KArgs& base, const StageLists& L, hipStream_t s, hipError_t* err, hipEvent_t* ev = nullptr);
constexpr int kStages = 5;
// Per-slice device counter block: the step counter (int at offset 0) and its snapshot
// (int kSnapWord).
constexpr size_t kCounterBytes = 256;
static_assert(kCounterBytes >= (kSnapWord + 1) * sizeof(int), "counter block holds the snapshot");

vp_status hip_status(hipError_t e, const char* what);
vp_status check_options(const vp_plan* p, const vp_options* o);

// The captured steps of a fit: a graph of one step and one of kMany. Between two graphs the GPU
// idles for 5 to 8 us (static 64^2: 27 us of kernels in a step of 32 us), between the kernels of one
// for none; eight steps a graph leave 1 us a step, and every count of steps is a few graphs.
// Capturing the larger graph takes the host 0.2 ms (64^2) to 0.9 ms (blade-aligned), what it gains
// in 50 to 200 steps. It is therefore captured behind kLead single steps, which keep the GPU busy
// meanwhile, by a call of twice as many, or of kMany once a fit in shorter calls has replayed kLong.
// First call of a new fit, one step a graph / the larger graph captured before the first step /
// behind the lead, ms: 64^2 x 40 steps 1.47 / 1.38 / 1.41, x 100 3.41 / 3.01 / 3.08, 256^2 x 40 4.06 /
// 4.14 / 3.88, blade-aligned 256^2 x 40 8.37 / 8.56 / 8.15, K-Planes 192^2 x 40 46.4 / 47.6 / 46.5.
struct StepGraph {
    static constexpr int kMany = 8, kLead = 2 * kMany, kLong = 16 * kMany;
    hipGraph_t graph[2] = {nullptr, nullptr};
    hipGraphExec_t exec[2] = {nullptr, nullptr};
    int64_t replayed = 0;
    ~StepGraph() { drop(); }
    void drop() {
        for (int i = 0; i < 2; ++i) {
            if (exec[i]) (void)hipGraphExecDestroy(exec[i]);
            if (graph[i]) (void)hipGraphDestroy(graph[i]);
            exec[i] = nullptr;
            graph[i] = nullptr;
        }
        replayed = 0;
    }
    // n steps on the stream; step() enqueues one (hipError_t).
    template <typename F>
    hipError_t run(hipStream_t s, int n, F step) {
        hipError_t e = hipSuccess;
        int left = n;
        auto singles = [&](int k) {
            if (k > 0 && !exec[0]) e = capture(s, 0, 1, step);
            for (; e == hipSuccess && k > 0; --k, --left) e = hipGraphLaunch(exec[0], s);
        };
        if (!exec[1] && (n >= 2 * kLead || (n >= kMany && replayed >= kLong))) {
            singles(std::min(left, kLead));
            if (e == hipSuccess) e = capture(s, 1, kMany, step);
        }
        if (exec[1])
            for (; e == hipSuccess && left >= kMany; left -= kMany) e = hipGraphLaunch(exec[1], s);
        if (e == hipSuccess) singles(left);
        replayed += n;
        return e;
    }

  private:
    template <typename F>
    hipError_t capture(hipStream_t s, int which, int steps, F step) {
        hipError_t e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess) return e;
        for (int i = 0; i < steps && e == hipSuccess; ++i) e = step();
        const hipError_t ce = hipStreamEndCapture(s, &graph[which]);
        if (e == hipSuccess) e = ce;
        if (e == hipSuccess) e = hipGraphInstantiate(&exec[which], graph[which], nullptr, nullptr, 0);
        if (e != hipSuccess && graph[which]) {
            (void)hipGraphDestroy(graph[which]);
            graph[which] = nullptr;
        }
        return e;
    }
};

}  // namespace vp

struct vp_session {
    const vp_plan* plan = nullptr;
    vp_options opts{};
    int device = -1;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    vp::DeviceTables* tabs = nullptr;
    const vp::Layout* layout = nullptr;
    const vp::DeviceLayout* dlayout = nullptr;
    bool own_shape = false;  // the layout's shape is the plan's own: neither asked for nor tuned
    float2* vol[2] = {nullptr, nullptr};
    float2* m = nullptr;
    float2* v = nullptr;
    float2* work = nullptr;
    float2* y = nullptr;
    float* loss_part = nullptr;
    int* step_dev = nullptr;
    double* dpart = nullptr;
    float2* render = nullptr;
    float2* grad = nullptr;  // data gradient, allocated when a separate update pass runs
    void* h_part = nullptr;  // pinned objective partials (doubles, then loss floats)
    int64_t steps_done = 0;
    vp::StepGraph graph;
    vp::SliceDesc desc{};
    vp::StageLists lists{};
    ~vp_session();
};

namespace vp {

// Device-resident group of slices sharing one stream: descriptors, concatenated work
// lists and (optionally) a captured step. Used by batched reconstructions and the server.
struct SliceGroup {
    int device = -1;
    hipStream_t stream = nullptr;
    SliceDesc* d_descs = nullptr;
    Task* d_tasks = nullptr;
    size_t cap_descs = 0, cap_tasks = 0;  // device capacities (grow only)
    std::vector<SliceDesc> h_descs;       // host copies, kept until the stream has read them
    std::vector<Task> h_tasks;
    StageLists lists{};
    StepGraph graph;
    ~SliceGroup();
};
// Builds descriptors and concatenated work lists for `sessions` (slice i = sessions[i],
// stopping at limits[i] steps) and enqueues their upload on the group's stream (no
// wait); drops any captured graph. Call it only once the stream has passed the previous
// upload (the host copies are reused).
vp_status group_build(SliceGroup* g, const std::vector<vp_session*>& sessions, const std::vector<int>& limits);
// Enqueues n_steps steps of every slice of the group (use_graph: replay captured steps).
vp_status group_run(SliceGroup* g, int n_steps, bool use_graph);

// Allocates and uploads a session on `stream` (nullptr: a stream of its own). The initial
// state is enqueued on `upload` (nullptr: the session stream) and waited for if `wait`;
// otherwise the caller keeps kspace and init alive until that stream has passed them.
vp_status session_alloc(const vp_plan* p, const vp_options* o, const vp_c64* kspace, const vp_c64* init,
                        hipStream_t stream, vp_session** out, hipStream_t upload = nullptr, bool wait = true);
vp_status session_run(vp_session* s, int32_t n_steps, int32_t use_graph);
// Allocates the session's data-gradient buffer (for a separate update pass) if missing.
vp_status session_ensure_grad(vp_session* s);
vp_status session_objective(vp_session* s, double* objective, double* data_term);
// The objective in two halves: kernels and pinned read-back enqueued on `stream`, then
// (after the caller has synchronised that stream) the host reduction.
vp_status session_objective_enqueue(vp_session* s, hipStream_t stream);
vp_status session_objective_finish(vp_session* s, double* objective, double* data_term);
vp_status session_read(vp_session* s, vp_c64* volume_out, vp_c64* proj_out, vp_c64* water_out, vp_c64* fat_out);
}  // namespace vp
