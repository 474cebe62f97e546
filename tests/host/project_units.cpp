// The projection kernel that a launch chooses, by the alignment of its volume: the launch functions are
// this program's, so nothing runs. Prints, for each region size, the variants chosen for a volume on
// 16 bytes, for one on 8, and for an odd n.
#include <cstdio>

#include "plan.h"
#include "runtime.h"

static const void* g_kernel;
static dim3 g_grid, g_block;
static size_t g_lds;

extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t) {
    g_grid = grid;
    g_block = block;
    g_lds = lds;
    return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
    *grid = g_grid;
    *block = g_block;
    *lds = g_lds;
    *s = nullptr;
    return hipSuccess;
}
extern "C" hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t) {
    g_kernel = f;
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }

int main() {
    int bad = 0;
    for (int waves : {4, 8})
        for (int re : {300, 512, 600, 1024, 1100, 2048, 2049, 4096}) {
            const void* kernel[4];
            size_t lds[4];
            for (int i = 0; i < 4; ++i) {
                vp::KArgs a{};
                a.ntasks = 1;
                // 16 bytes; 8 bytes; the second volume of a resumed step on 8 bytes; an odd n
                a.one.vol[0] = (float2*)(size_t)(i == 1 ? 0x10008 : 0x10000);
                a.one.vol[1] = (float2*)(size_t)(i == 2 ? 0x20008 : 0);
                if (vp::launch_project(a, 4, 1, waves, re, i == 3, nullptr) != hipSuccess) return 2;
                kernel[i] = g_kernel;
                lds[i] = g_lds;
            }
            const bool ok = kernel[1] == kernel[3] && kernel[2] == kernel[3] && lds[1] == lds[3] && lds[2] == lds[3] &&
                            (re > 2048 || kernel[0] != kernel[3]);
            bad += !ok;
            printf("waves %d region %d: %s\n", waves, re, ok ? "ok" : "16-byte units on 8 bytes");
        }
    return bad ? 1 : 0;
}
