// Evaluation kernels (Section 6): the coverage-weighted k-space average behind the
// baseline reconstructions, and the per-image terms of PSNR on magnitudes.

#include <type_traits>

#include "kcommon.h"

namespace vp {

constexpr int kAvgBlades = 5;  // the dynamic baseline's window

// Frame slot f of the launch is frame first + f: the average, over the blades
// max(0, first + f - window + 1) .. first + f that measure a sample, of their values
// there (ascending blade order), times 1/n, the unitary scale of the n x n inverse DFT
// that follows. Unmeasured samples are zero. window <= 0 takes every blade up to the frame.
// A thread takes V neighbouring pixels (V = 2 where n is even), the masks of kAvgBlades blades
// in flight together, then the values that they let through.
template <int V>
__global__ __launch_bounds__(kThreads) void k_baseline_avg(const uint8_t* __restrict__ mask,
                                                           const float2* __restrict__ y, float2* __restrict__ out,
                                                           int n, int window, int first) {
    const size_t nn = (size_t)n * n;
    const size_t px = ((size_t)blockIdx.x * kThreads + threadIdx.x) * V;
    if (px >= nn) return;
    const int f = first + (int)blockIdx.y;
    const int lo = window > 0 ? max(0, f - window + 1) : 0;
    using Mk = typename std::conditional<V == 2, uint16_t, uint8_t>::type;
    float2 acc[V];
    int c[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        acc[v] = make_float2(0.f, 0.f);
        c[v] = 0;
    }
    for (int b0 = lo; b0 <= f; b0 += kAvgBlades) {
        Mk on[kAvgBlades];
        float2 val[kAvgBlades][V];
#pragma unroll
        for (int k = 0; k < kAvgBlades; ++k) {
            on[k] = *reinterpret_cast<const Mk*>(mask + (size_t)min(b0 + k, f) * nn + px);
            if (b0 + k > f) on[k] = 0;
        }
#pragma unroll
        for (int k = 0; k < kAvgBlades; ++k) {
            if (on[k] != 0) {
#pragma unroll
                for (int v = 0; v < V; ++v) val[k][v] = y[(size_t)(b0 + k) * nn + px + v];
            }
        }
#pragma unroll
        for (int k = 0; k < kAvgBlades; ++k) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                if ((on[k] >> (8 * v)) & 0xff) {
                    acc[v] = cadd(acc[v], val[k][v]);
                    ++c[v];
                }
            }
        }
    }
#pragma unroll
    for (int v = 0; v < V; ++v)
        out[(size_t)blockIdx.y * nn + px + v] = cscale(acc[v], 1.0f / ((float)max(c[v], 1) * (float)n));
}

// Square root of x >= 0 in FP64: the hardware's FP32 reciprocal square root (about 1 ulp), a Newton
// step of the root and of its reciprocal (2^-46 relative), then a correction by the exact residual in
// FP64. What is rounded at the end is off by 2^-39 of an ulp: none of six million magnitudes differs
// from the correctly rounded one (one in a million does with the unrefined reciprocal in the
// correction). About half the library root's instructions, which bound k_psnr: one CU works on an
// image (16 frames of 192^2 through vp_psnr: 18.9 us, 21.0 us with the library's root; 384^2: 63 and 72 us).
// Values outside FP32's normal range take the library's.
__device__ __forceinline__ double sqrt64(double x) {
    const float xf = (float)x;
    if (!(xf >= 1.1754944e-38f && xf <= 3.4028235e38f)) return x == 0.0 ? 0.0 : sqrt(x);
    const double y = (double)__builtin_amdgcn_rsqf(xf);
    const double h0 = 0.5 * y, g = x * y, r = fma(-h0, g, 0.5);
    const double h = fma(h0, r, h0), s = fma(g, r, g);
    return fma(fma(-s, s, x), h, s);
}

// One block per image of npx samples: FP64 sum of (|image| - |truth|)^2 and the peak
// |truth|, reduced in a fixed order; terms[3 i + {0, 1, 2}] = mean squared error, peak,
// 10 log10(peak^2 / mse) (+inf for mse = 0).
constexpr int kPsnrThreads = 1024;
constexpr int kPsnrPer = 4;

__global__ __launch_bounds__(kPsnrThreads) void k_psnr(const float2* __restrict__ img,
                                                       const float2* __restrict__ truth, long long npx,
                                                       double* __restrict__ terms) {
    __shared__ double se[kPsnrThreads];
    __shared__ double pk[kPsnrThreads];
    const size_t off = (size_t)blockIdx.x * (size_t)npx;
    double e = 0.0, m = 0.0;
    // kPsnrPer samples of a thread in flight together, added in order
    for (long long i0 = threadIdx.x; i0 < npx; i0 += kPsnrPer * kPsnrThreads) {
        float2 a[kPsnrPer], t[kPsnrPer];
#pragma unroll
        for (int k = 0; k < kPsnrPer; ++k) {
            const long long i = min(i0 + (long long)k * kPsnrThreads, npx - 1);
            a[k] = img[off + i];
            t[k] = truth[off + i];
        }
#pragma unroll
        for (int k = 0; k < kPsnrPer; ++k) {
            if (i0 + (long long)k * kPsnrThreads < npx) {
                const double a2 = fma((double)a[k].x, (double)a[k].x, (double)a[k].y * a[k].y);
                const double t2 = fma((double)t[k].x, (double)t[k].x, (double)t[k].y * t[k].y);
                const double d = sqrt64(a2) - sqrt64(t2);
                e = fma(d, d, e);
                m = fmax(m, t2);
            }
        }
    }
    se[threadIdx.x] = e;
    pk[threadIdx.x] = m;
    __syncthreads();
    for (int h = kPsnrThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            se[threadIdx.x] += se[threadIdx.x + h];
            pk[threadIdx.x] = fmax(pk[threadIdx.x], pk[threadIdx.x + h]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double mse = se[0] / (double)npx, peak = sqrt(pk[0]);
        terms[3 * (size_t)blockIdx.x + 0] = mse;
        terms[3 * (size_t)blockIdx.x + 1] = peak;
        terms[3 * (size_t)blockIdx.x + 2] = mse > 0.0 ? 10.0 * log10(peak * peak / mse) : __builtin_inf();
    }
}

hipError_t launch_baseline_avg(const uint8_t* mask, const float2* y, float2* out, int n, int window, int first,
                               int n_frames, hipStream_t s) {
    if (n_frames <= 0) return hipSuccess;
    const size_t nn = (size_t)n * n;
    const size_t px = nn % 2 == 0 ? 2 * kThreads : kThreads;
    const dim3 g((unsigned)((nn + px - 1) / px), (unsigned)n_frames);
    if (nn % 2 == 0) hipLaunchKernelGGL(k_baseline_avg<2>, g, dim3(kThreads), 0, s, mask, y, out, n, window, first);
    else hipLaunchKernelGGL(k_baseline_avg<1>, g, dim3(kThreads), 0, s, mask, y, out, n, window, first);
    return hipGetLastError();
}

hipError_t launch_psnr(const float2* img, const float2* truth, long long npx, int n_images, double* terms,
                       hipStream_t s) {
    if (n_images <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_psnr, dim3((unsigned)n_images), dim3(kPsnrThreads), 0, s, img, truth, npx, terms);
    return hipGetLastError();
}

}  // namespace vp
