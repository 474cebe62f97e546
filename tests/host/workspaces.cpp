// Workspaces kept by a plan, with this program's memory, stream and event functions in place of
// the runtime's: which calls allocate, and how much stays allocated. Streams are small integers;
// work enqueued on one is finished when `finish` says so.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>

#include "plan.h"

using vp::Workspace;
using vp::WorkspaceSlots;

static std::map<void*, size_t> g_alive;           // allocations
static std::set<std::pair<size_t, size_t>> g_run; // (stream, event) recorded and not finished
static int g_mallocs, g_capturing = -1, g_relaxed, g_unsafe;

extern "C" {
hipError_t hipMallocAsync(void** p, size_t bytes, hipStream_t) {
    *p = malloc(1);
    g_alive[*p] = bytes;
    ++g_mallocs;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (!g_alive.erase(p)) abort();
    free(p);
    return hipSuccess;
}
hipError_t hipFreeAsync(void* p, hipStream_t) { return hipFree(p); }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c) {
    *c = (int)(size_t)s == g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) {
    for (auto it = g_run.begin(); it != g_run.end();)
        it = it->second == (size_t)e ? g_run.erase(it) : std::next(it);
    free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { g_run.insert({(size_t)s, (size_t)e}); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) {
    g_unsafe += !g_relaxed;  // would invalidate another thread's capture
    for (const auto& r : g_run)
        if (r.second == (size_t)e) return hipErrorNotReady;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
    const int was = g_relaxed;
    g_relaxed = *m == hipStreamCaptureModeRelaxed;
    *m = was ? hipStreamCaptureModeRelaxed : hipStreamCaptureModeGlobal;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
}

static hipStream_t stream(size_t i) { return (hipStream_t)(i + 16); }
static void finish(size_t i) {
    for (auto it = g_run.begin(); it != g_run.end();)
        it = it->first == i + 16 ? g_run.erase(it) : std::next(it);
}
static size_t kept() {
    size_t b = 0;
    for (const auto& a : g_alive) b += a.second;
    return b;
}
// A call with these workspaces at once, of `a` and (where not 0) `b` bytes; its allocations.
static int call(WorkspaceSlots* slots, size_t i, size_t a, size_t b = 0) {
    const int before = g_mallocs;
    Workspace x, y;
    if (x.take(slots, a, stream(i)) != hipSuccess || (b && y.take(slots, b, stream(i)) != hipSuccess)) exit(2);
    if (b && x.ptr == y.ptr) { printf("one workspace twice\n"); exit(2); }
    return g_mallocs - before;
}

int main(int, char**) {
    int bad = 0;
    char what[64];
    auto expect = [&](const char* name, size_t got, size_t want) {
        if (got == want) return;
        ++bad;
        printf("%s: %zu, not %zu\n", name, got, want);
    };
    if (scanf("%63s", what) != 1) return 2;
    const size_t MB = 1 << 20;
    if (!strcmp(what, "sizes")) {
        WorkspaceSlots s;  // a small and a large workspace per call, on one stream
        expect("first call", call(&s, 0, 1 * MB, 40 * MB), 2);
        for (int k = 0; k < 5; ++k) expect("later call", call(&s, 0, 1 * MB, 40 * MB), 0);
        expect("bytes kept", kept(), 41 * MB);
        expect("small call", call(&s, 0, 1 * MB), 0);
        expect("large call", call(&s, 0, 40 * MB), 0);
        expect("bytes kept", kept(), 41 * MB);
    } else if (!strcmp(what, "streams")) {
        {
            WorkspaceSlots s;  // streams that come and go
            for (size_t i = 0; i < 4; ++i) expect("first streams", call(&s, i, 2 * MB), 1);
            for (size_t i = 0; i < 4; ++i) finish(i);
            for (size_t i = 4; i < 12; ++i) {
                expect("a new stream takes a finished one's", call(&s, i, 2 * MB), 0);
                expect("and keeps it", call(&s, i, 2 * MB), 0);
                finish(i);
            }
            expect("bytes kept", kept(), 8 * MB);
        }
        expect("bytes kept by a plan that is gone", kept(), 0);
        {
            WorkspaceSlots s;  // all four at work: a fifth stream has memory of its own
            for (size_t i = 0; i < 4; ++i) call(&s, i, 2 * MB);
            expect("fifth stream", call(&s, 4, 2 * MB), 1);
            expect("bytes kept", kept(), 8 * MB);
            finish(2);  // one finished: its slot goes over, replaced where it is too small
            expect("larger call", call(&s, 4, 6 * MB), 1);
            expect("again", call(&s, 4, 6 * MB), 0);
            expect("bytes kept", kept(), 12 * MB);
            for (size_t i : {0, 1, 3}) expect("the others keep theirs", call(&s, i, 2 * MB), 0);
        }
        {
            WorkspaceSlots s;  // one stream whose calls grow
            for (size_t k = 1; k <= 10; ++k) {
                expect("a larger call", call(&s, 0, k * MB), 1);
                finish(0);
                expect("again", call(&s, 0, k * MB), 0);
                finish(0);
            }
            if (kept() > 40 * MB) expect("bytes kept", kept(), 40 * MB);
        }
        expect("queries outside relaxed mode", g_unsafe, 0);
        expect("mode left relaxed", g_relaxed, 0);
    } else if (!strcmp(what, "own")) {
        WorkspaceSlots s;  // captured streams, the per-thread default stream and large calls keep nothing
        call(&s, 0, 2 * MB);
        expect("kept", kept(), 2 * MB);
        g_capturing = 16;
        for (int k = 0; k < 2; ++k) expect("captured", call(&s, 0, 2 * MB), 1);
        g_capturing = -1;
        for (int k = 0; k < 2; ++k) {
            const int before = g_mallocs;
            Workspace x;
            if (x.take(&s, 2 * MB, hipStreamPerThread) != hipSuccess) return 2;
            expect("per thread", g_mallocs - before, 1);
        }
        for (int k = 0; k < 2; ++k) expect("large", call(&s, 0, 65 * MB), 1);
        expect("kept", kept(), 2 * MB);
        expect("slot again", call(&s, 0, 2 * MB), 0);
    } else {
        return 2;
    }
    printf("%d bad\n", bad);
    return bad ? 1 : 0;
}
