// StepGraph's schedule of captures and launches, with this program's graph functions in place of
// the runtime's. For every sequence of calls: each call runs exactly its steps, and the larger graph
// is captured only where its rule says, behind steps that are already enqueued.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "runtime.h"

using vp::StepGraph;

static int g_steps;      // steps recorded in the open capture
static int g_ran;        // steps launched in this call
static int g_instances;  // executable graphs alive
static std::vector<int> g_captured;  // sizes captured in this call, and what had been launched before
static std::vector<int> g_before;

extern "C" {
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { g_steps = 0; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = (hipGraph_t)malloc(1); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    int* x = (int*)malloc(sizeof(int));
    *x = g_steps;
    *e = (hipGraphExec_t)x;
    ++g_instances;
    g_captured.push_back(g_steps);
    g_before.push_back(g_ran);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) { g_ran += *(int*)e; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { free(e); --g_instances; return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { free(g); return hipSuccess; }
}

int main() {
    int bad = 0;
    auto check = [&](bool ok, const char* what, const std::vector<int>& calls) {
        if (ok) return;
        ++bad;
        printf("%s in calls", what);
        for (int n : calls) printf(" %d", n);
        printf("\n");
    };
    std::vector<std::vector<int>> sequences;
    for (int n = 1; n <= 300; ++n) sequences.push_back({n});
    for (int n : {1, 2, 5, 7, 8, 9, 15, 16, 17, 20, 31}) sequences.push_back(std::vector<int>(300 / n + 2, n));
    sequences.push_back({5, 20});
    sequences.push_back({40, 3, 8, 1, 100});
    for (const auto& calls : sequences) {
        {
            StepGraph g;
            int done = 0;
            bool large = false;
            for (int n : calls) {
                g_ran = 0;
                g_captured.clear();
                g_before.clear();
                const hipError_t e = g.run(nullptr, n, [] { ++g_steps; return hipSuccess; });
                check(e == hipSuccess && g_ran == n, "steps lost or added", calls);
                bool now = false;
                for (size_t i = 0; i < g_captured.size(); ++i) {
                    check(g_captured[i] == 1 || g_captured[i] == StepGraph::kMany, "a graph of another size", calls);
                    if (g_captured[i] != StepGraph::kMany) continue;
                    check(!large && !now, "the larger graph twice", calls);
                    now = true;
                    // the host's work on it is hidden behind steps, and pays within the call or by
                    // the length of the fit so far
                    check(g_before[i] >= StepGraph::kMany, "the larger graph ahead of the steps", calls);
                    check(n >= 32 || done >= 128, "the larger graph in a short fit", calls);
                }
                large = large || now;
                done += n;
                check(large || n < 32, "a long call without the larger graph", calls);
            }
            check(large || done < 128 + 2 * calls[0] || calls[0] < StepGraph::kMany, "a long fit without it", calls);
        }
        check(g_instances == 0, "graphs left", calls);
    }
    printf("%zu sequences, %d bad\n", sequences.size(), bad);
    return bad ? 1 : 0;
}
