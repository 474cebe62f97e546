// Voxel-wise kernels: operator TV/L1 gradient, objective regulariser terms and the
// renders (Section 4.3, Section 6 fat/water split).

#include <algorithm>

#include "kcommon.h"

namespace vp {

// ------------------------------------------------------------------ voxel-wise kernels

// Operator TV/L1 gradient: grad (+)= tv_w grad TV + l1_w grad L1 (weights from the descriptor).
// A block takes kTvPx pixels of one bin's plane (blockIdx.y = knot * S + bin), the planes and rows
// around them served by the caches; all loads of a thread's pixels are issued before any is used
// (a missing neighbour reads the pixel itself and is not added). It is bound by those cache
// loads; with a 64-bit division per coordinate of every voxel it was bound by them instead
// (150^2 x 12 bins x 5 knots: 49 us, now 11.6 us).
constexpr int kTvPer = 2;
constexpr int kTvPx = kTvPer * kThreads;
__global__ __launch_bounds__(kThreads) void k_tv_grad(const float2* __restrict__ V, float2* __restrict__ grad, int n,
                                                      int S, int T, float tv_w, float l1_w, float teps, int accumulate) {
    const float eps2 = charb_eps2(teps), ninv = 1.0f / (float)n;
    const int nn = n * n;
    const bool tv = tv_w != 0.f, l1 = l1_w != 0.f;
    for (int plane = blockIdx.y; plane < S * T; plane += gridDim.y) {
        const int t = plane / S, s = plane - t * S;
        const size_t p0 = (size_t)plane * nn;
        float2 v0[kTvPer], nb[kTvPer][8], old[kTvPer];
        int px[kTvPer], xx[kTvPer], yy[kTvPer];
#pragma unroll
        for (int k = 0; k < kTvPer; ++k) {
            const int p = blockIdx.x * kTvPx + k * kThreads + threadIdx.x;
            px[k] = p;
            const int q = min(p, nn - 1);
            const int y = small_div(q, ninv), x = q - y * n;
            xx[k] = x;
            yy[k] = y;
            const size_t i = p0 + q;
            v0[k] = V[i];
            if (tv) {
                nb[k][0] = V[t > 0 ? i - (size_t)S * nn : i];
                nb[k][1] = V[t + 1 < T ? i + (size_t)S * nn : i];
                nb[k][2] = V[s > 0 ? i - nn : i];
                nb[k][3] = V[s + 1 < S ? i + nn : i];
                nb[k][4] = V[y > 0 ? i - n : i];
                nb[k][5] = V[y + 1 < n ? i + n : i];
                nb[k][6] = V[x > 0 ? i - 1 : i];
                nb[k][7] = V[x + 1 < n ? i + 1 : i];
            }
            if (accumulate) old[k] = grad[i];
        }
#pragma unroll
        for (int k = 0; k < kTvPer; ++k) {
            if (px[k] >= nn) continue;
            float2 g = make_float2(0.f, 0.f);
            if (tv) {
                if (t > 0) g = cadd(g, charb_w(csub(v0[k], nb[k][0]), eps2));
                if (t + 1 < T) g = csub(g, charb_w(csub(nb[k][1], v0[k]), eps2));
                if (s > 0) g = cadd(g, charb_w(csub(v0[k], nb[k][2]), eps2));
                if (s + 1 < S) g = csub(g, charb_w(csub(nb[k][3], v0[k]), eps2));
                if (yy[k] > 0) g = cadd(g, charb_w(csub(v0[k], nb[k][4]), eps2));
                if (yy[k] + 1 < n) g = csub(g, charb_w(csub(nb[k][5], v0[k]), eps2));
                if (xx[k] > 0) g = cadd(g, charb_w(csub(v0[k], nb[k][6]), eps2));
                if (xx[k] + 1 < n) g = csub(g, charb_w(csub(nb[k][7], v0[k]), eps2));
                g = cscale(g, tv_w);
            }
            if (l1) g = cfma(l1_w, charb_w(v0[k], eps2), g);
            if (accumulate) g = cadd(old[k], g);
            grad[p0 + px[k]] = g;
        }
    }
}

// Objective regulariser terms: per work item, sums of the TV terms (forward differences
// where the neighbour exists) and the L1 terms, each written as |z|^2 / (sqrt(|z|^2 + e^2) + e),
// the cancellation-free form of sqrt(|z|^2 + e^2) - e. Output a.dpart[2 * item + {0, 1}].
__global__ __launch_bounds__(kThreads) void k_reg_value(const KArgs a) {
    __shared__ double red[2][kThreads];
    for (int ti = blockIdx.x; ti < a.ntasks; ti += gridDim.x) {
        const AS4 Task* tk = cst(a.tasks) + ti;
        const int slice = tk->slice;
        int* const stepp = DF(step);
        const int st = read_step(stepp);
        const int n = DF(n), S = DF(S), T = DF(T);
        const size_t nn = (size_t)n * n, nvox = (size_t)T * S * nn;
        const size_t i0 = (size_t)tk->a * kVoxItem;
        const float2* V = stepp ? DF(vol[st & 1]) : DF(vol[0]);
        const float e = DF(tv_eps), e2 = e * e;
        double tv = 0.0, l1 = 0.0;
        // the item's first plane (knot * S + bin) and offset in it; a voxel's plane, row and column
        // follow by 32-bit arithmetic
        const int q0 = (int)(i0 / nn), r0 = (int)(i0 - (size_t)q0 * nn);
        const float nninv = 1.0f / (float)(n * n), ninv = 1.0f / (float)n;
        const int cnt = (int)min(nvox - i0, (size_t)kVoxItem);
        for (int j = threadIdx.x; j < cnt; j += kThreads) {
            const size_t i = i0 + j;
            const int dq = small_div(r0 + j, nninv), p = r0 + j - dq * (n * n);
            const int y = small_div(p, ninv), x = p - y * n;
            const int t = (q0 + dq) / S, s = q0 + dq - t * S;
            const float2 v0 = V[i];
            float part = 0.f;
            auto term = [&](float2 z) {
                const float q = __builtin_fmaf(z.x, z.x, z.y * z.y);
                return q / (sqrtf(q + e2) + e);
            };
            if (x + 1 < n) part += term(csub(V[i + 1], v0));
            if (y + 1 < n) part += term(csub(V[i + n], v0));
            if (s + 1 < S) part += term(csub(V[i + nn], v0));
            if (t + 1 < T) part += term(csub(V[i + (size_t)S * nn], v0));
            tv += part;
            l1 += term(v0);
        }
        red[0][threadIdx.x] = tv;
        red[1][threadIdx.x] = l1;
        __syncthreads();
        for (int w = kThreads / 2; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) {
                red[0][threadIdx.x] += red[0][threadIdx.x + w];
                red[1][threadIdx.x] += red[1][threadIdx.x + w];
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            a.dpart[2 * ti] = red[0][0];
            a.dpart[2 * ti + 1] = red[1][0];
        }
        __syncthreads();
    }
}

// Render at phi = 0 and the fat/water split: water = bins [0, split), fat = [split, S),
// proj = water + fat. One work item per (knot, block of kVoxItem pixels).
__global__ __launch_bounds__(kThreads) void k_render(const KArgs a) {
    for (int ti = blockIdx.x; ti < a.ntasks; ti += gridDim.x) {
        const AS4 Task* tk = cst(a.tasks) + ti;
        const int slice = tk->slice;
        int* const stepp = DF(step);
        const int st = read_step(stepp);
        const int n = DF(n), S = DF(S);
        const size_t nn = (size_t)n * n;
        const int split = a.split_bin < 0 ? S / 2 : min(a.split_bin, S);
        const float2* V = (stepp ? DF(vol[st & 1]) : DF(vol[0])) + (size_t)tk->a * S * nn;
        const size_t p0 = (size_t)tk->b * kVoxItem;
        for (size_t p = p0 + threadIdx.x; p < min(nn, p0 + kVoxItem); p += blockDim.x) {
            float2 w = make_float2(0.f, 0.f), f = make_float2(0.f, 0.f);
            for (int s = 0; s < split; ++s) w = cadd(w, V[(size_t)s * nn + p]);
            for (int s = split; s < S; ++s) f = cadd(f, V[(size_t)s * nn + p]);
            const size_t o = (size_t)tk->a * nn + p;
            if (a.out0) a.out0[o] = cadd(w, f);
            if (a.out1) a.out1[o] = w;
            if (a.out2) a.out2[o] = f;
        }
    }
}

// ------------------------------------------------------------------ launchers

static inline int grid_for(int ntasks) { return ntasks < 1 ? 1 : (ntasks > (1 << 20) ? (1 << 20) : ntasks); }

hipError_t launch_tv_grad(const KArgs& a, hipStream_t s) {
    const SliceDesc& d = a.one;
    const dim3 g((unsigned)((d.n * d.n + kTvPx - 1) / kTvPx), (unsigned)std::min(d.S * d.T, 65535));
    hipLaunchKernelGGL(k_tv_grad, g, dim3(kThreads), 0, s, d.vol[0], d.grad, d.n, d.S, d.T, d.tv_w, d.l1_w, d.tv_eps,
                       a.accumulate);
    return hipGetLastError();
}
hipError_t launch_reg_value(const KArgs& a, hipStream_t s) {
    if (a.ntasks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_reg_value, dim3(grid_for(a.ntasks)), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}
hipError_t launch_render(const KArgs& a, hipStream_t s) {
    if (a.ntasks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_render, dim3(grid_for(a.ntasks)), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace vp
