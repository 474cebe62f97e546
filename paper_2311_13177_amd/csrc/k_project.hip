// Sheared spectral projection (Section 4.2 "Projection").

#include <algorithm>

#include "kcommon.h"

namespace vp {

// ------------------------------------------------------------------ projection
//
// P_b[y][x] = sum_s sum_taps w * V_s[y + oy + (0|1)][x + ox + (0|1)]   (Section 4.2)
// Work item: (part group, tile row, tile column), tile = 64 columns x PPT rows, NW waves
// (4 or 8) sharing the staged volume regions. Part e of the group belongs to wave
// e % NW, slot e / NW. Each lane owns one column and accumulates PPT rows for each of
// its GW parts over the bins in ascending order.

// The planes go from memory straight to LDS in a ring of D phases of P planes (pb bytes each),
// D - 1 phases in flight, with one barrier per phase. LDS reads (9 cycles of a CU per row of a
// part and bin) and the taps' arithmetic (8 cycles over its four SIMDs) bound it, then, where
// the volume streams from HBM, its bytes. They overlap only between waves: staging without
// registers leaves the kernel at 24 to 40 VGPRs and exact plane sizes fit three or more
// eight-wave blocks on a CU. Measured (192^2 x 32 bins x 16 knots, 12 rows): 55 us with planes
// staged through registers two phases deep, 43 us so; 256^2 x 32 bins, 12 parts: 34 and 20 us.
// A software pipeline of the LDS reads (100 to 130 VGPRs, half the waves) was slower, as were
// taps held in the lanes and reading the planes through the vector cache without LDS.
template <int GW, int PPT, int SE, int P, int D, int UB, int NW>
__global__ __launch_bounds__(64 * NW) void k_project(const KArgs a, int pb) {
    extern __shared__ float2 sm[];
    using Sg = DmaStager<SE, UB, 64 * NW>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (a.snap) step_snapshot(a);
    for (int ti = xcd_item(blockIdx.x, gridDim.x); ti < a.ntasks; ti += gridDim.x) {
        const AS4 Task* tk = cst(a.tasks) + ti;
        const int slice = tk->slice;
        int* const stepp = DF(step);
        const int st = read_step(stepp);
        if (stepp && st >= DF(step_limit)) continue;
        const int n = DF(n), S = DF(S), B = DF(B), nparts = DF(nparts), sched = DF(schedule);
        const unsigned sseed = DF(sched_seed);
        const size_t nn = (size_t)n * n;
        const AS4 ProjGroup* gr = cst(DF(groups)) + tk->a;
        const int knot = gr->knot, ge0 = gr->e0, gne = gr->ne;
        // (16-byte units: from an even column, an even number of columns)
        const int oxmin = UB == 16 ? gr->ox_min & ~1 : gr->ox_min, oymin = gr->oy_min;
        const int RH = PPT + gr->oy_max - oymin + 1;
        const int RW = UB == 16 ? (kTileW + gr->ox_max - oxmin + 2) & ~1 : kTileW + gr->ox_max - oxmin + 1;
        const int y0 = tk->b * PPT, x0 = tk->c * kTileW;
        const AS4 KnotEntry* ent = cst(DF(knot_ent));
        const AS4 ShearEntry* shear = cst(DF(shear));
        float2* const work = DF(work);
        const float2* const V = (stepp ? DF(vol[st & 1]) : DF(vol[0])) + (size_t)knot * S * nn;
        int eb[GW], ep[GW];
        bool act[GW];
#pragma unroll
        for (int j = 0; j < GW; ++j) {
            const int e = j * NW + wave;
            act[j] = false;
            eb[j] = 0;
            ep[j] = 0;
            if (e < gne) {
                eb[j] = ent[ge0 + e].blade;
                ep[j] = ent[ge0 + e].part;
                act[j] = active_blade(sched, sseed, stepp, st, B, eb[j]);
            }
        }
        float2 acc[GW][PPT];
#pragma unroll
        for (int j = 0; j < GW; ++j)
#pragma unroll
            for (int i = 0; i < PPT; ++i) acc[j][i] = make_float2(0.f, 0.f);
        Sg sg;
        sg.init(RH, RW, y0 + oymin, x0 + oxmin, n, pb);
        const int phase = P * pb;
        auto issue = [&](int s0, int slot) {
#pragma unroll
            for (int p = 0; p < P; ++p)
                sg.issue(s0 + p < S ? V + (size_t)(s0 + p) * nn : nullptr, (int)nn, slot * phase + p * pb);
        };
#pragma unroll
        for (int d = 0; d < D - 1; ++d) issue(d * P, d);
        int slot = 0;
        for (int s0 = 0; s0 < S; s0 += P) {
            // this phase has landed for every wave, and every wave is done with the one before,
            // whose slot takes the phase D - 1 ahead
            sg.template wait<(D - 2) * P>();
            issue(s0 + (D - 1) * P, slot == 0 ? D - 1 : slot - 1);
            const float2* buf = sm + slot * (phase / 8);
            slot = slot + 1 == D ? 0 : slot + 1;
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int s = s0 + p;
                if (s < S) {
#pragma unroll
                    for (int j = 0; j < GW; ++j) {
                        if (act[j]) {
                            const AS4 ShearEntry* sh = shear + eb[j] * S + s;
                            const float w00 = sh->w00, w01 = sh->w01, w10 = sh->w10, w11 = sh->w11;
                            const float2* L = buf + p * (pb / 8) + (sh->oy - oymin) * RW + (sh->ox - oxmin) + lane;
                            float2 a0 = L[0], a1 = L[1];
#pragma unroll
                            for (int i = 0; i < PPT; ++i) {
                                const float2 b0 = L[(i + 1) * RW], b1 = L[(i + 1) * RW + 1];
                                float2 t = acc[j][i];
                                t = cfma(w00, a0, t);
                                t = cfma(w01, a1, t);
                                t = cfma(w10, b0, t);
                                t = cfma(w11, b1, t);
                                acc[j][i] = t;
                                a0 = b0;
                                a1 = b1;
                            }
                        }
                    }
                }
            }
        }
        sg.template wait<0>();  // nothing of this item lands in the LDS of the next
        const int x = x0 + lane;
#pragma unroll
        for (int j = 0; j < GW; ++j) {
            if (act[j] && x < n) {
                float2* out = work + ((size_t)eb[j] * nparts + ep[j]) * nn;
#pragma unroll
                for (int i = 0; i < PPT; ++i) {
                    const int y = y0 + i;
                    if (y < n) out[(size_t)y * n + x] = acc[j][i];
                }
            }
        }
    }
}

// ------------------------------------------------------------------ launchers

static inline int grid_for(int ntasks) { return ntasks < 1 ? 1 : (ntasks > (1 << 20) ? (1 << 20) : ntasks); }

// Units per thread, planes per phase and phases of the ring (at most 64 KiB) follow the largest
// region of the launch. narrow: 4-byte units (an odd n, or a volume that is not on 16 bytes).
template <int GW, int PPT, int NW>
static void project_variant(const KArgs& a, int re, bool narrow, hipStream_t s) {
    const dim3 g(grid_for(a.ntasks)), b(64 * NW);
    constexpr int W = 8 / NW;
    // a plane's LDS bytes: whole chunks of a wave's units, at least as many as SE asks for
    auto plane = [&](int se, int ub) { return std::max((re * 8 + 64 * ub - 1) / (64 * ub), (se - 1) * NW + 1) * 64 * ub; };
#define PL(SE, P, D, UB)                                                                           \
    do {                                                                                           \
        const int pb = plane(SE, UB);                                                              \
        hipLaunchKernelGGL((k_project<GW, PPT, SE, P, D, UB, NW>), g, b, (D) * (P) * pb, s, a, pb); \
    } while (0)
    if (re > 2048) PL(16 * W, 1, 2, 4);
    else if (narrow && re > 1024) PL(8 * W, 1, 3, 4);
    else if (narrow) PL(4 * W, 1, 4, 4);
    else if (re > 1024) PL(2 * W, 1, 3, 16);
    else if (NW == 4 && re <= 512) PL(1, 2, 2, 16);
    else PL(W, 2, 2, 16);
#undef PL
}

hipError_t launch_project(const KArgs& a, int rows, int gw, int waves, int re, bool odd, hipStream_t s) {
    if (a.ntasks <= 0) return hipSuccess;
    if (!proj_tiles_ok(rows, gw) || !item_waves_ok(waves) || re < 1 || re > kStageMax * kThreads)
        return hipErrorInvalidValue;
    // a caller's volume is on 8 bytes; a descriptor array's are allocations of the sessions
    const bool narrow = odd || (!a.descs && (((uintptr_t)a.one.vol[0] | (uintptr_t)a.one.vol[1]) & 15) != 0);
#define PV(R, G)                                                            \
    case R * 16 + G:                                                        \
        if constexpr (proj_tiles_ok(R, G)) {                                \
            if (waves == 8) project_variant<G, R, 8>(a, re, narrow, s);     \
            else project_variant<G, R, 4>(a, re, narrow, s);                \
        }                                                                   \
        break
    switch (rows * 16 + gw) {
        PV(1, 1); PV(1, 2); PV(1, 4); PV(1, 8);
        PV(2, 1); PV(2, 2); PV(2, 4); PV(2, 8);
        PV(4, 1); PV(4, 2); PV(4, 4);
        PV(8, 1); PV(8, 2); PV(12, 1);
        default: return hipErrorInvalidValue;
    }
#undef PV
    return hipGetLastError();
}

}  // namespace vp
