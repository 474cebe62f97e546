// Kernels of the complex K-Planes dynamic model (Section 4.1): the separable factors,
// the dense per-blade decode, the gradient back through the factors (gather form, fixed
// summation orders), the grid regularisers of Section 4.3 and the optimiser update.

#include "kcommon.h"
#include "kplanes.h"

namespace vp {

namespace {

// a * b + c and conj(a) * b + c with explicit fused multiply-adds
__device__ __forceinline__ float2 cmad(float2 a, float2 b, float2 c) {
    return make_float2(__builtin_fmaf(a.x, b.x, __builtin_fmaf(-a.y, b.y, c.x)),
                       __builtin_fmaf(a.x, b.y, __builtin_fmaf(a.y, b.x, c.y)));
}
__device__ __forceinline__ float2 cjmad(float2 a, float2 b, float2 c) {
    return make_float2(__builtin_fmaf(a.x, b.x, __builtin_fmaf(a.y, b.y, c.x)),
                       __builtin_fmaf(a.x, b.y, __builtin_fmaf(-a.y, b.x, c.y)));
}
// (1 - w) a + w b
__device__ __forceinline__ float2 clerp(float2 a, float2 b, float w) { return cfma(w, b, cscale(a, 1.0f - w)); }

typedef float f32v4 __attribute__((ext_vector_type(4)));

// Indices are split by 32-bit divisions; a fit's element counts fit 31 bits (2 scales x 256 bins x
// 256 blades x 512 samples x 16 features is the most). The kernels over a decode's times, whose
// number is the caller's, are compiled for 64 bits too (Ix).
__device__ __forceinline__ unsigned gtid() { return blockIdx.x * blockDim.x + threadIdx.x; }
__device__ __forceinline__ unsigned gstride() { return gridDim.x * blockDim.x; }

// Feature-planar arrays (Z, Zt, XA) hold row r's features in pairs (single with F = 1): feature f
// of sample i at ((r (F / P) + f / P) n + i) P + f % P, P = min(F, 2). A wave of 64 samples then
// reads 16 contiguous bytes per lane, one access for two features.
__device__ __forceinline__ int feat_pair(int F) { return F > 1 ? 2 : 1; }
template <int F>
__device__ __forceinline__ void load_planar(float2 (&o)[F], const float2* row, int n, int i) {
    if constexpr (F == 1) {
        o[0] = row[i];
    } else {
#pragma unroll
        for (int u = 0; u < F / 2; ++u) {
            const float4 q = *reinterpret_cast<const float4*>(row + 2 * ((size_t)u * n + i));
            o[2 * u] = make_float2(q.x, q.y);
            o[2 * u + 1] = make_float2(q.z, q.w);
        }
    }
}
// One sample's features in a row of [n][F], the same for the whole wave (scalar loads).
template <int F>
__device__ __forceinline__ void load_uniform(float2 (&o)[F], const float2* p) {
    typedef float vec __attribute__((ext_vector_type(2 * (F > 8 ? 8 : F))));
    constexpr int FV = F > 8 ? 8 : F;
#pragma unroll
    for (int u = 0; u < F / FV; ++u) {
        const vec q = *cst(reinterpret_cast<const vec*>(p + u * FV));
#pragma unroll
        for (int f = 0; f < FV; ++f) o[u * FV + f] = make_float2(q[2 * f], q[2 * f + 1]);
    }
}

// Grid value of scale c along one spatial axis at sample i: p[stride * node] rows.
__device__ __forceinline__ float2 read_x(const float2* p, long long stride, const KPDesc& d, int c, int i) {
    const int i0 = d.nd0[c * d.n + i];
    const int i1 = min(i0 + 1, d.R[c] - 1);
    return clerp(p[i0 * stride], p[i1 * stride], d.ndw[c * d.n + i]);
}

// ------------------------------------------------------------------ factors

// Xs, Ys [ns][S][n][F]
__global__ __launch_bounds__(kThreads) void k_kp_fac_s(const KPDesc d) {
    const unsigned total = (unsigned)d.ns * d.S * d.n * d.F;
    for (unsigned e = gtid(); e < total; e += gstride()) {
        const int f = (int)(e % d.F);
        const int i = (int)((e / d.F) % d.n);
        const int s = (int)((e / ((unsigned)d.F * d.n)) % d.S);
        const int c = (int)(e / ((unsigned)d.F * d.n * d.S));
        const int R = d.R[c];
        const float2* xs = d.params + d.off[c][KP_XS] + (long long)s * R * d.F + f;
        const float2* ys = d.params + d.off[c][KP_YS] + (long long)s * R * d.F + f;
        d.Xs[e] = read_x(xs, d.F, d, c, i);
        d.Ys[e] = read_x(ys, d.F, d, c, i);
    }
}

// qx, qy [ns][B][n][F] and qs [ns][B][S][F]: time grids at each time
template <typename Ix>
__global__ __launch_bounds__(kThreads) void k_kp_fac_t(const KPDesc d) {
    const Ix nq = (Ix)d.ns * d.B * d.n * d.F;
    const Ix total = nq + (Ix)d.ns * d.B * d.S * d.F;
    for (Ix e = gtid(); e < total; e += gstride()) {
        if (e < nq) {
            const int f = (int)(e % d.F);
            const int i = (int)((e / d.F) % d.n);
            const int b = (int)((e / ((Ix)d.F * d.n)) % d.B);
            const int c = (int)(e / ((Ix)d.F * d.n * d.B));
            const int R = d.R[c];
            const int k0 = d.tk[b], k1 = min(k0 + 1, d.Rt - 1);
            const float a = d.ta[b];
            const float2* xt = d.params + d.off[c][KP_XT] + f;
            const float2* yt = d.params + d.off[c][KP_YT] + f;
            const long long row = (long long)R * d.F;
            d.qx[e] = clerp(read_x(xt + k0 * row, d.F, d, c, i), read_x(xt + k1 * row, d.F, d, c, i), a);
            d.qy[e] = clerp(read_x(yt + k0 * row, d.F, d, c, i), read_x(yt + k1 * row, d.F, d, c, i), a);
        } else {
            const Ix r = e - nq;
            const int f = (int)(r % d.F);
            const int s = (int)((r / d.F) % d.S);
            const int b = (int)((r / ((Ix)d.F * d.S)) % d.B);
            const int c = (int)(r / ((Ix)d.F * d.S * d.B));
            const int k0 = d.tk[b], k1 = min(k0 + 1, d.Rt - 1);
            const float2* st = d.params + d.off[c][KP_ST] + (long long)s * d.F + f;
            const long long row = (long long)d.S * d.F;
            d.qs[r] = clerp(st[k0 * row], st[k1 * row], d.ta[b]);
        }
    }
}

// Z: the xy grid at (y, x), along x first, feature-planar with rows y; Zt the same values with
// rows x (each written in its own order)
__global__ __launch_bounds__(kThreads) void k_kp_fac_z(const KPDesc d) {
    const unsigned per = (unsigned)d.ns * d.n * d.n * d.F, P = feat_pair(d.F);
    const unsigned total = d.Zt ? 2 * per : per;
    for (unsigned e = gtid(); e < total; e += gstride()) {
        const bool tr = e >= per;
        const unsigned q = tr ? e - per : e;
        const int i = (int)((q / P) % d.n);
        const unsigned ru = q / (P * d.n);  // row and feature pair
        const int f = (int)((ru % (d.F / P)) * P + q % P);
        const int r = (int)((ru / (d.F / P)) % d.n);
        const int c = (int)(ru / (d.F / P) / d.n);
        const int x = tr ? r : i, y = tr ? i : r;
        const int R = d.R[c];
        const float2* xy = d.params + d.off[c][KP_XY] + f;
        const int j0 = d.nd0[c * d.n + y], j1 = min(j0 + 1, R - 1);
        const float2 r0 = read_x(xy + (long long)j0 * R * d.F, d.F, d, c, x);
        const float2 r1 = read_x(xy + (long long)j1 * R * d.F, d.F, d, c, x);
        (tr ? d.Zt : d.Z)[q] = clerp(r0, r1, d.ndw[c * d.n + y]);
    }
}

// XA = a Xs qx qs, [ns][B][S] rows feature-planar, the same as [ns][B][S][n][F] (XAt), and
// Yf = Ys qy, [ns][B][S][n][F]
template <typename Ix>
__global__ __launch_bounds__(kThreads) void k_kp_prod(const KPDesc d) {
    const Ix total = (Ix)d.ns * d.B * d.S * d.n * d.F;
    const unsigned P = feat_pair(d.F), FN = (Ix)d.F * d.n;
    for (Ix e = gtid(); e < total; e += gstride()) {
        const Ix row = e / FN;
        const unsigned in = (unsigned)(e - row * FN);  // row (c, b, s)
        const Ix cb = row / d.S, s = row - cb * d.S;
        const Ix cs = cb / d.B * d.S + s;
        auto xa = [&](unsigned i, unsigned f) {
            return cmul(cmul(cmul(d.params[d.a_off + f], d.Xs[cs * FN + i * d.F + f]), d.qx[cb * FN + i * d.F + f]),
                        d.qs[row * d.F + f]);
        };
        const unsigned u = in / (P * d.n);
        d.XA[e] = xa(in / P - u * d.n, u * P + in % P);
        if (d.XAt) d.XAt[e] = xa(in / d.F, in % d.F);
        d.Yf[e] = cmul(d.Ys[cs * FN + in], d.qy[cb * FN + in]);
    }
}

// ------------------------------------------------------------------ decode

// vol[b][s][y][x] = sum_c sum_f Z[c][y][x][f] XA[c][b][s][x][f] Yf[c][b][s][y][f]
//
// A wave task is (blade, kDecBins bins, kDecRows rows, 64 columns): its XA values (per
// column) are loaded once for all kDecRows rows, its Yf values (per row, the same in
// every lane) by scalar loads, and Z (per pixel) once per row for all kDecBins bins. A block's
// four waves take two neighbouring row groups by two bin groups, so that each value read is
// used by two waves of the CU, and the blocks of an XCD share rows (their Z stays in its L2).
// The sums run in the same order as a per-voxel loop (scales, then features), so every shape
// of this task gives the same bits. Its FP32 operations are the bound (8 per voxel, feature
// and scale: 123 us at the full clock for 32 blades x 32 bins x 192^2, 8 features, 2 scales;
// 195 us taken in a fit, 232 with four bins a wave, where half the waves fit).
constexpr int kDecBins = 2;
constexpr int kDecRows = 4;

template <int F>
__global__ __launch_bounds__(kThreads) void k_kp_decode(const KPDesc d) {
    const int n = d.n, S = d.S;
    const long long nn = (long long)n * n;
    const int sqp = (S + 2 * kDecBins - 1) / (2 * kDecBins);
    const int nseg = (n + 63) / 64, nrp = (n + 2 * kDecRows - 1) / (2 * kDecRows);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned W = (unsigned)d.B * sqp * nrp * nseg;
    for (unsigned w = xcd_item(blockIdx.x, gridDim.x); w < W; w += gridDim.x) {
        const int qp = w % sqp, b = (w / sqp) % d.B, sg = w / ((unsigned)sqp * d.B);
        const int seg = sg % nseg, rp = sg / nseg;
        const int s0 = (qp * 2 + (wave >> 1)) * kDecBins, ns = min(kDecBins, S - s0);
        const int y0 = (rp * 2 + (wave & 1)) * kDecRows;
        if (ns <= 0 || y0 >= n) continue;
        const int x = seg * 64 + lane;
        const int xs = min(x, n - 1);
        float2 v[kDecRows][kDecBins];
#pragma unroll
        for (int r = 0; r < kDecRows; ++r)
#pragma unroll
            for (int k = 0; k < kDecBins; ++k) v[r][k] = make_float2(0.f, 0.f);
        for (int c = 0; c < d.ns; ++c) {
            const long long cb = ((long long)c * d.B + b) * S + s0;
            float2 xa[kDecBins][F];
#pragma unroll
            for (int k = 0; k < kDecBins; ++k) load_planar<F>(xa[k], d.XA + (cb + min(k, ns - 1)) * n * F, n, xs);
#pragma unroll
            for (int r = 0; r < kDecRows; ++r) {
                const int y = min(y0 + r, n - 1);
                float2 z[F];
                load_planar<F>(z, d.Z + ((long long)c * n + y) * n * F, n, xs);
#pragma unroll
                for (int k = 0; k < kDecBins; ++k) {
                    float2 yf[F];
                    load_uniform<F>(yf, d.Yf + ((cb + min(k, ns - 1)) * n + y) * F);
#pragma unroll
                    for (int f = 0; f < F; ++f) v[r][k] = cmad(cmul(z[f], xa[k][f]), yf[f], v[r][k]);
                }
            }
        }
        if (x < n) {
#pragma unroll
            for (int r = 0; r < kDecRows; ++r)
#pragma unroll
                for (int k = 0; k < kDecBins; ++k)
                    if (k < ns && y0 + r < n) d.vol[((long long)b * S + s0 + k) * nn + (long long)(y0 + r) * n + x] = v[r][k];
        }
    }
}

// ------------------------------------------------------------------ gradient through the factors

// gZ[c][y][x][f] = sum_b sum_s conj(XA Yf) G[b][s][y][x], in two passes: partial sums over
// consecutive (b, s) chunks for every pixel and both scales (G read once), then the
// chunks summed in order. A wave task of the first pass is (chunk, kGzRows rows, 64
// columns): each XA value (per column) serves all kGzRows rows, the Yf values (per row, the
// same in every lane) are scalar loads, and a block's four waves take neighbouring rows of
// one chunk, so that XA comes from the CU's cache for three of them. Each sum runs over
// (b, s) in order. Bound by its FP32 operations (123 us at the sizes above; 200 us, 296 with
// XA as [n][F], four waves a block without a value in common and a last round of few blocks).
constexpr int kGzRows = 2;

template <int F>
__global__ __launch_bounds__(kThreads) void k_kp_grad_z(const KPDesc d) {
    const int n = d.n;
    const long long nn = (long long)n * n;
    const int nbs = d.B * d.S, cs = (nbs + d.zchunks - 1) / d.zchunks;
    const int nseg = (n + 63) / 64, nrb = (n + 4 * kGzRows - 1) / (4 * kGzRows);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int W = d.zchunks * nrb * nseg;
    for (int w = xcd_item(blockIdx.x, gridDim.x); w < W; w += gridDim.x) {
        const int y0 = ((w % nrb) * 4 + wave) * kGzRows;
        const int seg = (w / nrb) % nseg, ch = w / (nrb * nseg);
        if (y0 >= n) continue;
        const int x = seg * 64 + lane;
        const int xs = min(x, n - 1);
        float2 acc[kGzRows][kKpMaxScales][F];
#pragma unroll
        for (int r = 0; r < kGzRows; ++r)
#pragma unroll
            for (int c = 0; c < kKpMaxScales; ++c)
#pragma unroll
                for (int f = 0; f < F; ++f) acc[r][c][f] = make_float2(0.f, 0.f);
        const int bs1 = min(nbs, (ch + 1) * cs);
        for (int bs = ch * cs; bs < bs1; ++bs) {
            float2 g[kGzRows];
#pragma unroll
            for (int r = 0; r < kGzRows; ++r) g[r] = d.G[(long long)bs * nn + (long long)min(y0 + r, n - 1) * n + xs];
#pragma unroll
            for (int c = 0; c < kKpMaxScales; ++c) {
                if (c < d.ns) {
                    const long long cb = (long long)c * nbs + bs;
                    float2 xa[F];
                    load_planar<F>(xa, d.XA + cb * n * F, n, xs);
#pragma unroll
                    for (int r = 0; r < kGzRows; ++r) {
                        float2 yf[F];
                        load_uniform<F>(yf, d.Yf + (cb * n + min(y0 + r, n - 1)) * F);
#pragma unroll
                        for (int f = 0; f < F; ++f) acc[r][c][f] = cjmad(cmul(xa[f], yf[f]), g[r], acc[r][c][f]);
                    }
                }
            }
        }
        if (x < n) {
#pragma unroll
            for (int r = 0; r < kGzRows; ++r) {
#pragma unroll
                for (int c = 0; c < kKpMaxScales; ++c) {
                    if (c < d.ns && y0 + r < n) {
                        float2* out = d.zpart + (((long long)ch * d.ns + c) * nn + (long long)(y0 + r) * n + x) * F;
#pragma unroll
                        for (int f = 0; f < F; ++f) out[f] = acc[r][c][f];
                    }
                }
            }
        }
    }
}

__global__ __launch_bounds__(kThreads) void k_kp_grad_z_sum(const KPDesc d) {
    const unsigned per = (unsigned)d.ns * d.n * d.n * d.F;
    for (unsigned e = gtid(); e < per; e += gstride()) {
        float2 acc = make_float2(0.f, 0.f);
        for (int ch = 0; ch < d.zchunks; ++ch) acc = cadd(acc, d.zpart[(size_t)ch * per + e]);
        d.gZ[e] = acc;
    }
}

// gXA[c][b][s][x][f] = sum_y conj(Z Yf) G[b][s][y][x] and gY[c][b][s][y][f] =
// sum_x conj(Z XA) G[b][s][y][x]: the same sum with the axes exchanged. A wave task is
// (BS consecutive (b, s), 64 lanes along one axis, one of PARTS parts of the other axis): each Z
// (Zt) value serves all BS (b, s) and both scales' sums read G once; the other factor is the
// same in every lane (scalar loads). A block is one task: its PARTS waves' sums, each in order, are
// added through LDS. Bound by its FP32 operations (123 us at the sizes above; gXA 205 us, 296 with
// G read once per scale, the halves summed by a kernel of their own and Z as [n][F]).
//
// Two (b, s) a wave by eight parts (four for gY) halve the loads of Z; one by eight has twice the
// waves. The second is taken below kGxWaves tasks of one (b, s) (two by eight parts against
// one by eight, gXA with 8 features: 1024 tasks of 256^2 96 and 144 us, 512 of 128^2 21 and 19 us, 256 of
// 256^2 63 and 53 us) and with 16 features, whose sums of two leave room for two waves per SIMD (3072 of
// 192^2: 588 and 508 us).
constexpr int kGxWaves = 1024;
constexpr int kGxParts = 8, kGyParts = 4, kWideParts = 8;
inline bool kp_one_bs(const KPDesc& d) {
    return d.F > 8 || (long long)d.B * d.S * ((d.n + 63) / 64) < kGxWaves;
}

// The waves of parts 1.. leave their sums in LDS, one scale at a time, and the first part's
// wave adds them to its own in order and stores (lane `at` of row c nbs + bs of [n][F]).
template <int F, int BS, int PARTS>
__device__ __forceinline__ void add_parts(float2* red, const float2 (&acc)[BS][kKpMaxScales][F], int part, int lane,
                                          float2* out, int ns, int nbs, int bs0, int n, int at) {
    constexpr int kOne = BS * F * 64;
    float2* const mine = red + lane;
#pragma unroll
    for (int c = 0; c < kKpMaxScales; ++c) {
        if (c < ns) {
            __syncthreads();
            if (part > 0) {
#pragma unroll
                for (int j = 0; j < BS; ++j)
#pragma unroll
                    for (int f = 0; f < F; ++f) mine[(part - 1) * kOne + (j * F + f) * 64] = acc[j][c][f];
            }
            __syncthreads();
            if (part == 0 && at < n) {
#pragma unroll
                for (int j = 0; j < BS; ++j) {
                    if (bs0 + j < nbs) {
                        float2* o = out + (((long long)c * nbs + bs0 + j) * n + at) * F;
#pragma unroll
                        for (int f = 0; f < F; ++f) {
                            float2 v = acc[j][c][f];
#pragma unroll
                            for (int q = 0; q < PARTS - 1; ++q) v = cadd(v, mine[q * kOne + (j * F + f) * 64]);
                            o[f] = v;
                        }
                    }
                }
            }
        }
    }
}

template <int F, int BS, int PARTS>
__global__ __launch_bounds__(64 * PARTS) void k_kp_grad_x(const KPDesc d) {
    __shared__ float2 red[(PARTS - 1) * BS * F * 64];
    const int n = d.n;
    const long long nn = (long long)n * n;
    const int nbs = d.B * d.S, ntp = (nbs + BS - 1) / BS;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int W = ntp * ((n + 63) / 64), rq = (n + PARTS - 1) / PARTS;
    for (int w = xcd_item(blockIdx.x, gridDim.x); w < W; w += gridDim.x) {
        const int bs0 = (w % ntp) * BS;
        const int x = (w / ntp) * 64 + lane, xs = min(x, n - 1);
        const int ya = wave * rq, yb = bs0 < nbs ? min(n, ya + rq) : 0;
        float2 acc[BS][kKpMaxScales][F];
#pragma unroll
        for (int j = 0; j < BS; ++j)
#pragma unroll
            for (int c = 0; c < kKpMaxScales; ++c)
#pragma unroll
                for (int f = 0; f < F; ++f) acc[j][c][f] = make_float2(0.f, 0.f);
        for (int y = ya; y < yb; ++y) {
            float2 g[BS];
#pragma unroll
            for (int j = 0; j < BS; ++j) g[j] = d.G[(long long)min(bs0 + j, nbs - 1) * nn + (long long)y * n + xs];
#pragma unroll
            for (int c = 0; c < kKpMaxScales; ++c) {
                if (c < d.ns) {
                    float2 z[F];
                    load_planar<F>(z, d.Z + ((long long)c * n + y) * n * F, n, xs);
#pragma unroll
                    for (int j = 0; j < BS; ++j) {
                        float2 yf[F];
                        load_uniform<F>(yf, d.Yf + (((long long)c * nbs + min(bs0 + j, nbs - 1)) * n + y) * F);
#pragma unroll
                        for (int f = 0; f < F; ++f) acc[j][c][f] = cjmad(cmul(z[f], yf[f]), g[j], acc[j][c][f]);
                    }
                }
            }
        }
        add_parts<F, BS, PARTS>(red, acc, wave, lane, d.gXA, d.ns, nbs, bs0, n, x);
    }
}

// The lanes run over y here, so a wave turns its part of G (64 rows by kGyCols columns of each of
// its (b, s)) through its own LDS: a lane loads 16 bytes of a row, four lanes a row's 64 bytes,
// and reads back its own row; the 16-byte units of row r are permuted by (r / 4) % 4, which
// keeps both sides free of bank conflicts. (gY 200 us at the sizes above; 460 us with the lanes
// over x, two rows of Z and of XA loaded for four sums and 63 exchanges between lanes at the end.)
// The parts take groups of kGyCols columns in turn: they use the lines of G that one of them has
// brought in.
constexpr int kGyCols = 8;

// Orders the LDS accesses of a wave's lanes among themselves: the hardware runs a wave's in order,
// the fence keeps the compiler to it.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// PAIR: n is even and G on a 16-byte boundary, so that a lane's two columns are one access (a branch
// at run time was compiled into four loads for both cases: 277 us instead of 200).
template <int F, int BS, int PARTS, bool PAIR>
__global__ __launch_bounds__(64 * PARTS) void k_kp_grad_y(const KPDesc d) {
    constexpr int kTile = 64 * kGyCols;  // values of one (b, s)
    constexpr int kRed = (PARTS - 1) * BS * F * 64, kTiles = PARTS * BS * kTile;
    __shared__ __attribute__((aligned(16))) float2 red[kRed > kTiles ? kRed : kTiles];
    const int n = d.n;
    const long long nn = (long long)n * n;
    const int nbs = d.B * d.S, ntp = (nbs + BS - 1) / BS;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    f32v4* const tile = reinterpret_cast<f32v4*>(red + wave * BS * kTile);
    const int W = ntp * ((n + 63) / 64);
    for (int w = xcd_item(blockIdx.x, gridDim.x); w < W; w += gridDim.x) {
        const int bs0 = (w % ntp) * BS;
        const int y0 = (w / ntp) * 64;
        const int y = y0 + lane, ys = min(y, n - 1);
        const int xb = bs0 < nbs ? n : 0;
        float2 acc[BS][kKpMaxScales][F];
#pragma unroll
        for (int j = 0; j < BS; ++j)
#pragma unroll
            for (int c = 0; c < kKpMaxScales; ++c)
#pragma unroll
                for (int f = 0; f < F; ++f) acc[j][c][f] = make_float2(0.f, 0.f);
        __syncthreads();  // the sums of the item before are read from the tiles' memory
        for (int x0 = wave * kGyCols; x0 < xb; x0 += PARTS * kGyCols) {
            f32v4 t[BS][4];
#pragma unroll
            for (int j = 0; j < BS; ++j) {
                const float2* G = d.G + (long long)min(bs0 + j, nbs - 1) * nn;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float2* row = G + (long long)min(y0 + i * 16 + lane / 4, n - 1) * n;
                    const int xc = x0 + 2 * (lane % 4);
                    if constexpr (PAIR) {
                        t[j][i] = *reinterpret_cast<const f32v4*>(row + min(xc, n - 2));
                    } else {
                        const float2 p = row[min(xc, n - 1)], q = row[min(xc + 1, n - 1)];
                        t[j][i] = f32v4{p.x, p.y, q.x, q.y};
                    }
                }
            }
            wave_lds_order();
#pragma unroll
            for (int j = 0; j < BS; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    tile[j * (kTile / 2) + (i * 16 + lane / 4) * 4 + ((lane % 4) ^ (lane / 16))] = t[j][i];
            wave_lds_order();
            const int xe = min(x0 + kGyCols, xb);
#pragma unroll 1
            for (int x = x0; x < xe; ++x) {
                const int q = (x - x0) / 2, h = (x - x0) % 2;
                float2 g[BS];
#pragma unroll
                for (int j = 0; j < BS; ++j)
                    g[j] = reinterpret_cast<const float2*>(tile)[2 * (j * (kTile / 2) + lane * 4 + (q ^ ((lane / 4) % 4))) + h];
#pragma unroll
                for (int c = 0; c < kKpMaxScales; ++c) {
                    if (c < d.ns) {
                        float2 z[F];
                        load_planar<F>(z, d.Zt + ((long long)c * n + x) * n * F, n, ys);
#pragma unroll
                        for (int j = 0; j < BS; ++j) {
                            float2 xv[F];
                            load_uniform<F>(xv, d.XAt + (((long long)c * nbs + min(bs0 + j, nbs - 1)) * n + x) * F);
#pragma unroll
                            for (int f = 0; f < F; ++f) acc[j][c][f] = cjmad(cmul(z[f], xv[f]), g[j], acc[j][c][f]);
                        }
                    }
                }
            }
        }
        add_parts<F, BS, PARTS>(red, acc, wave, lane, d.gY, d.ns, nbs, bs0, n, y);
    }
}

// ------------------------------------------------------------------ chain to the grids

// Independent sums over one index each, a thread per output:
//   gXs[c][s][x][f] = sum_b conj(a qx qs) gXA        gqx[c][b][x][f] = sum_s conj(a Xs qs) gXA
//   gYs[c][s][y][f] = sum_b conj(qy) gY              gqy[c][b][y][f] = sum_s conj(Ys) gY
// (h and gqs, with far fewer outputs and a longer sum, are k_kp_chain_h's)
__global__ __launch_bounds__(kThreads) void k_kp_chain1(const KPDesc d) {
    const int n = d.n, S = d.S, B = d.B, F = d.F;
    const unsigned n_sn = (unsigned)d.ns * S * n * F;   // gXs, gYs
    const unsigned n_bn = (unsigned)d.ns * B * n * F;   // gqx, gqy
    const unsigned total = 2 * n_sn + 2 * n_bn;
    for (unsigned e = gtid(); e < total; e += gstride()) {
        float2 acc = make_float2(0.f, 0.f);
        if (e < 2 * n_sn) {
            const bool isx = e < n_sn;
            const unsigned r = isx ? e : e - n_sn;
            const int f = (int)(r % F);
            const int i = (int)((r / F) % n);
            const int s = (int)((r / ((unsigned)F * n)) % S);
            const int c = (int)(r / ((unsigned)F * n * S));
            const float2 a = d.params[d.a_off + f];
            for (int b = 0; b < B; ++b) {
                const long long cbs = ((long long)c * B + b) * S + s;
                const long long qi = (((long long)c * B + b) * n + i) * F + f;
                const float2 gv = (isx ? d.gXA : d.gY)[(cbs * n + i) * F + f];
                const float2 w = isx ? cmul(cmul(a, d.qx[qi]), d.qs[cbs * F + f]) : d.qy[qi];
                acc = cjmad(w, gv, acc);
            }
            (isx ? d.gXs : d.gYs)[r] = acc;
        } else if (e < 2 * n_sn + 2 * n_bn) {
            const unsigned e2 = e - 2 * n_sn;
            const bool isx = e2 < n_bn;
            const unsigned r = isx ? e2 : e2 - n_bn;
            const int f = (int)(r % F);
            const int i = (int)((r / F) % n);
            const int b = (int)((r / ((unsigned)F * n)) % B);
            const int c = (int)(r / ((unsigned)F * n * B));
            const float2 a = d.params[d.a_off + f];
            for (int s = 0; s < S; ++s) {
                const long long cbs = ((long long)c * B + b) * S + s;
                const long long si = (((long long)c * S + s) * n + i) * F + f;
                const float2 gv = (isx ? d.gXA : d.gY)[(cbs * n + i) * F + f];
                const float2 w = isx ? cmul(cmul(a, d.Xs[si]), d.qs[cbs * F + f]) : d.Ys[si];
                acc = cjmad(w, gv, acc);
            }
            (isx ? d.gqx : d.gqy)[r] = acc;
        }
    }
}

// h[c][b][s][f] = sum_x conj(Xs qx) gXA and gqs = conj(a) h: a wave per output, lane l
// summing x = l, l + 64, ... in order, then the wave's 64 partial sums by a fixed
// butterfly (every lane ends with the same total)
__global__ __launch_bounds__(kThreads) void k_kp_chain_h(const KPDesc d) {
    const int n = d.n, S = d.S, B = d.B, F = d.F;
    const long long n_bs = (long long)d.ns * B * S * F;
    const int lane = threadIdx.x & 63;
    for (long long r = (long long)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); r < n_bs;
         r += (long long)gridDim.x * (kThreads / 64)) {
        const int f = (int)(r % F);
        const long long cbs = r / F;
        const int s = (int)(cbs % S);
        const int b = (int)((cbs / S) % B);
        const int c = (int)(cbs / ((long long)S * B));
        float2 acc = make_float2(0.f, 0.f);
        for (int x = lane; x < n; x += 64) {
            const float2 w = cmul(d.Xs[(((long long)c * S + s) * n + x) * F + f],
                                  d.qx[(((long long)c * B + b) * n + x) * F + f]);
            acc = cjmad(w, d.gXA[(cbs * n + x) * F + f], acc);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            acc.x += __shfl_xor(acc.x, o);
            acc.y += __shfl_xor(acc.y, o);
        }
        if (lane == 0) {
            d.h[r] = acc;
            d.gqs[r] = cjmad(d.params[d.a_off + f], acc, make_float2(0.f, 0.f));
        }
    }
}

// ga[f] = sum_c sum_b sum_s conj(qs) h: one block per feature, strided partial sums then
// a tree in a fixed order
__global__ __launch_bounds__(kThreads) void k_kp_chain_a(const KPDesc d) {
    __shared__ float2 red[kThreads];
    const int f = blockIdx.x;
    float2 acc = make_float2(0.f, 0.f);
    const long long nbs = (long long)d.ns * d.B * d.S;
    for (long long cbs = threadIdx.x; cbs < nbs; cbs += kThreads) acc = cjmad(d.qs[cbs * d.F + f], d.h[cbs * d.F + f], acc);
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int h = kThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] = cadd(red[threadIdx.x], red[threadIdx.x + h]);
        __syncthreads();
    }
    if (threadIdx.x == 0) d.ga[f] = red[0];
}

// Which grid holds flat element e, and its index within the grid (a: plane KP_PLANES).
__device__ __forceinline__ void locate(const KPDesc& d, long long e, int* c, int* pl, long long* idx) {
    if (e >= d.a_off) {
        *c = 0; *pl = KP_PLANES; *idx = e - d.a_off;
        return;
    }
    for (int cc = d.ns - 1; cc >= 0; --cc)
        for (int p = KP_PLANES - 1; p >= 0; --p)
            if (e >= d.off[cc][p]) {
                *c = cc; *pl = p; *idx = e - d.off[cc][p];
                return;
            }
    *c = 0; *pl = 0; *idx = e;
}

// Length of a grid's first and second axes (F is the third).
__device__ __forceinline__ void grid_dims(const KPDesc& d, int c, int pl, int* d0, int* d1) {
    const int R = d.R[c];
    switch (pl) {
        case KP_XY: *d0 = R; *d1 = R; break;
        case KP_XS: case KP_YS: *d0 = d.S; *d1 = R; break;
        case KP_XT: case KP_YT: *d0 = d.Rt; *d1 = R; break;
        default: *d0 = d.Rt; *d1 = d.S; break;
    }
}

// Grid regulariser gradient (Section 4.3 readings): Charbonnier TV along the grid's x, y
// and omega axes, squared second differences along t and Charbonnier sparsity of p - 1
// on the time grids.
__device__ float2 reg_grad(const KPDesc& d, int c, int pl, int i0, int i1, int f, const float2* p) {
    int d0, d1;
    grid_dims(d, c, pl, &d0, &d1);
    const long long s0 = (long long)d1 * d.F, s1 = d.F;  // strides of the two axes
    const float2 v = p[0];
    float2 g = make_float2(-0.f, -0.f);
    const bool time = pl == KP_XT || pl == KP_YT || pl == KP_ST;
    if (d.tv_w != 0.f) {
        float2 t = make_float2(-0.f, -0.f);
        if (!time) {  // axis 0 is x, y or omega for the static grids
            if (i0 > 0) t = cadd(t, charb_w(csub(v, p[-s0]), d.eps2));
            if (i0 + 1 < d0) t = csub(t, charb_w(csub(p[s0], v), d.eps2));
        }
        if (i1 > 0) t = cadd(t, charb_w(csub(v, p[-s1]), d.eps2));
        if (i1 + 1 < d1) t = csub(t, charb_w(csub(p[s1], v), d.eps2));
        g = cfma(d.tv_w, t, g);
    }
    if (time && d.smooth_w != 0.f) {
        // d2_m = p[m+1] - 2 p[m] + p[m-1], m in [1, d0 - 2]; p[k] appears in m = k-1, k, k+1
        float2 t = make_float2(-0.f, -0.f);
        for (int m = i0 - 1; m <= i0 + 1; ++m) {
            if (m < 1 || m > d0 - 2) continue;
            const float2* q = p + (long long)(m - i0) * s0;
            const float2 d2 = cadd(csub(q[s0], cscale(q[0], 2.f)), q[-s0]);
            const float coef = m == i0 ? -4.f : 2.f;
            t = cfma(coef, d2, t);
        }
        g = cfma(d.smooth_w, t, g);
    }
    if (time && d.sparse_w != 0.f) g = cfma(d.sparse_w, charb_w(make_float2(v.x - 1.f, v.y), d.eps2), g);
    return g;
}

// Data gradient of every grid element (transposed interpolation, gather form) plus the
// regulariser gradient -> grad.
__global__ __launch_bounds__(kThreads) void k_kp_grid(const KPDesc d) {
    const int n = d.n, S = d.S, F = d.F;
    for (unsigned e = gtid(); e < d.n_params; e += gstride()) {
        int c, pl;
        long long idx;
        locate(d, e, &c, &pl, &idx);
        if (pl == KP_PLANES) {
            d.grad[e] = d.ga[idx];
            continue;
        }
        int d0, d1;
        grid_dims(d, c, pl, &d0, &d1);
        const unsigned ix = (unsigned)idx;
        const int f = (int)(ix % F);
        const int i1 = (int)((ix / F) % d1);
        const int i0 = (int)(ix / ((unsigned)F * d1));
        const int* tp = d.tr_ptr + c * (n + 1);
        float2 acc = make_float2(0.f, 0.f);
        switch (pl) {
            case KP_XY:  // rows i0 (y nodes), columns i1 (x nodes)
                for (int a = tp[i0]; a < tp[i0 + 1]; ++a) {
                    const int y = d.tr_smp[a];
                    float2 row = make_float2(0.f, 0.f);
                    for (int q = tp[i1]; q < tp[i1 + 1]; ++q)
                        row = cfma(d.tr_w[q], d.gZ[(((long long)c * n + y) * n + d.tr_smp[q]) * F + f], row);
                    acc = cfma(d.tr_w[a], row, acc);
                }
                break;
            case KP_XS:
            case KP_YS: {
                const float2* src = pl == KP_XS ? d.gXs : d.gYs;
                for (int q = tp[i1]; q < tp[i1 + 1]; ++q)
                    acc = cfma(d.tr_w[q], src[(((long long)c * S + i0) * n + d.tr_smp[q]) * F + f], acc);
                break;
            }
            case KP_XT:
            case KP_YT: {
                const float2* src = pl == KP_XT ? d.gqx : d.gqy;
                for (int t = d.tt_ptr[i0]; t < d.tt_ptr[i0 + 1]; ++t) {
                    const int b = d.tt_b[t];
                    float2 part = make_float2(0.f, 0.f);
                    for (int q = tp[i1]; q < tp[i1 + 1]; ++q)
                        part = cfma(d.tr_w[q], src[(((long long)c * d.B + b) * n + d.tr_smp[q]) * F + f], part);
                    acc = cfma(d.tt_w[t], part, acc);
                }
                break;
            }
            default:  // omega-t: rows i0 (time nodes), columns i1 (bins)
                for (int t = d.tt_ptr[i0]; t < d.tt_ptr[i0 + 1]; ++t)
                    acc = cfma(d.tt_w[t], d.gqs[(((long long)c * d.B + d.tt_b[t]) * S + i1) * F + f], acc);
                break;
        }
        d.grad[e] = cadd(acc, reg_grad(d, c, pl, i0, i1, f, d.params + e));
    }
}

// Regulariser value: per element its forward differences (TV), the second difference
// centred on it (smoothness) and its sparsity term, as |z|^2 / (sqrt(|z|^2 + e^2) + e) for
// the Charbonnier terms; FP64 block sums in a fixed order -> rpart[block].
__global__ __launch_bounds__(kThreads) void k_kp_reg_value(const KPDesc d) {
    __shared__ double red[kThreads];
    const double e2 = (double)d.eps2, ep = sqrt(e2);
    auto charb = [&](float2 z) {
        const double q = (double)z.x * z.x + (double)z.y * z.y;
        return q / (sqrt(q + e2) + ep);
    };
    double acc = 0.0;
    for (unsigned e = gtid(); e < d.a_off; e += gstride()) {
        int c, pl;
        long long idx;
        locate(d, e, &c, &pl, &idx);
        int d0, d1;
        grid_dims(d, c, pl, &d0, &d1);
        const unsigned ix = (unsigned)idx;
        const int i1 = (int)((ix / d.F) % d1);
        const int i0 = (int)(ix / ((unsigned)d.F * d1));
        const long long s0 = (long long)d1 * d.F, s1 = d.F;
        const float2* p = d.params + e;
        const bool time = pl == KP_XT || pl == KP_YT || pl == KP_ST;
        if (d.tv_w != 0.f) {
            double t = 0.0;
            if (!time && i0 + 1 < d0) t += charb(csub(p[s0], p[0]));
            if (i1 + 1 < d1) t += charb(csub(p[s1], p[0]));
            acc += (double)d.tv_w * t;
        }
        if (time && d.smooth_w != 0.f && i0 >= 1 && i0 <= d0 - 2) {
            const double rx = ((double)p[s0].x - 2.0 * p[0].x) + p[-s0].x;
            const double ry = ((double)p[s0].y - 2.0 * p[0].y) + p[-s0].y;
            acc += (double)d.smooth_w * (rx * rx + ry * ry);
        }
        if (time && d.sparse_w != 0.f) acc += (double)d.sparse_w * charb(make_float2(p[0].x - 1.f, p[0].y));
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int h = kThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) d.rpart[blockIdx.x] = red[0];
}

// Adam (or GD) on every parameter, (Re, Im) as independent reals; step t = counter + 1.
__global__ __launch_bounds__(kThreads) void k_kp_update(const KPDesc d) {
    const int st = d.step ? *d.step : 0;
    const bool adam = d.optimizer == VP_OPT_ADAM;
    float step_size = d.lr, inv_bc2s = 1.f;
    if (adam) {
        const float tf = (float)(st + 1);
        const float bc1 = -expm1f(tf * d.ln_beta1), bc2 = -expm1f(tf * d.ln_beta2);
        step_size = d.lr / bc1;
        inv_bc2s = 1.f / sqrtf(bc2);
    }
    float2* p = const_cast<float2*>(d.params);
    for (unsigned e = gtid(); e < d.n_params; e += gstride()) {
        const float2 g = d.grad[e], v0 = p[e];
        if (adam) {
            float2 m = d.m[e], v = d.v[e];
            m.x = __builtin_fmaf(d.beta1, m.x, d.c1 * g.x);
            m.y = __builtin_fmaf(d.beta1, m.y, d.c1 * g.y);
            v.x = __builtin_fmaf(d.beta2, v.x, (d.c2 * g.x) * g.x);
            v.y = __builtin_fmaf(d.beta2, v.y, (d.c2 * g.y) * g.y);
            d.m[e] = m;
            d.v[e] = v;
            const float dx = __builtin_fmaf(__builtin_amdgcn_sqrtf(v.x), inv_bc2s, d.aeps);
            const float dy = __builtin_fmaf(__builtin_amdgcn_sqrtf(v.y), inv_bc2s, d.aeps);
            p[e] = make_float2(__builtin_fmaf(-step_size, m.x * __builtin_amdgcn_rcpf(dx), v0.x),
                               __builtin_fmaf(-step_size, m.y * __builtin_amdgcn_rcpf(dy), v0.y));
        } else {
            p[e] = make_float2(__builtin_fmaf(-d.lr, g.x, v0.x), __builtin_fmaf(-d.lr, g.y, v0.y));
        }
    }
}

__global__ void k_kp_advance(int* step) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *step = *step + 1;
}

// proj / water / fat of vol [B][S][n][n]
template <typename Ix>
__global__ __launch_bounds__(kThreads) void k_kp_render(const KPDesc d, int split, float2* proj, float2* water,
                                                        float2* fat) {
    const long long nn = (long long)d.n * d.n;
    const Ix total = (Ix)(d.B * nn);
    for (Ix e = gtid(); e < total; e += gstride()) {
        const Ix b = e / (Ix)nn, px = e % (Ix)nn;
        float2 w = make_float2(0.f, 0.f), ft = w;
        for (int s = 0; s < d.S; ++s) {
            const float2 v = d.vol[((long long)b * d.S + s) * nn + px];
            if (s < split) w = cadd(w, v);
            else ft = cadd(ft, v);
        }
        if (proj) proj[e] = cadd(w, ft);
        if (water) water[e] = w;
        if (fat) fat[e] = ft;
    }
}

// The kernel over `total` elements with the index type that they need.
#define KP_IX(KERNEL, TOTAL, ...)                                                                                   \
    if ((TOTAL) >> 31) hipLaunchKernelGGL(KERNEL<unsigned long long>, dim3(grid_of(TOTAL)), dim3(kThreads), 0, s, __VA_ARGS__); \
    else hipLaunchKernelGGL(KERNEL<unsigned>, dim3(grid_of(TOTAL)), dim3(kThreads), 0, s, __VA_ARGS__)

inline unsigned grid_of(long long total) {
    const long long g = (total + kThreads - 1) / kThreads;
    return (unsigned)(g < 1 ? 1 : (g > (1 << 20) ? (1 << 20) : g));
}

}  // namespace

bool kp_features_ok(int f) { return f == 1 || f == 2 || f == 4 || f == 8 || f == 16; }

hipError_t kp_launch_factors(const KPDesc& d, hipStream_t s) {
    const dim3 b(kThreads);
    hipLaunchKernelGGL(k_kp_fac_s, dim3(grid_of((long long)d.ns * d.S * d.n * d.F)), b, 0, s, d);
    const long long nt = (long long)d.ns * d.B * (d.n + d.S) * d.F, np = (long long)d.ns * d.B * d.S * d.n * d.F;
    KP_IX(k_kp_fac_t, nt, d);
    hipLaunchKernelGGL(k_kp_fac_z, dim3(grid_of((d.Zt ? 2LL : 1LL) * d.ns * d.n * d.n * d.F)), b, 0, s, d);
    KP_IX(k_kp_prod, np, d);
    return hipGetLastError();
}

#define KP_F_SWITCH(KERNEL, GRID)                                                   \
    switch (d.F) {                                                                  \
        case 1: hipLaunchKernelGGL(KERNEL<1>, GRID, dim3(kThreads), 0, s, d); break;   \
        case 2: hipLaunchKernelGGL(KERNEL<2>, GRID, dim3(kThreads), 0, s, d); break;   \
        case 4: hipLaunchKernelGGL(KERNEL<4>, GRID, dim3(kThreads), 0, s, d); break;   \
        case 8: hipLaunchKernelGGL(KERNEL<8>, GRID, dim3(kThreads), 0, s, d); break;   \
        case 16: hipLaunchKernelGGL(KERNEL<16>, GRID, dim3(kThreads), 0, s, d); break; \
        default: return hipErrorInvalidValue;                                       \
    }

inline unsigned blocks_of(long long items) { return (unsigned)(items > (1 << 20) ? (1 << 20) : items); }

hipError_t kp_launch_decode(const KPDesc& d, hipStream_t s) {
    const long long items = (long long)d.B * ((d.S + 2 * kDecBins - 1) / (2 * kDecBins)) *
                            ((d.n + 2 * kDecRows - 1) / (2 * kDecRows)) * ((d.n + 63) / 64);
    KP_F_SWITCH(k_kp_decode, dim3(blocks_of(items)));
    return hipGetLastError();
}

hipError_t kp_launch_back_z(const KPDesc& d, hipStream_t s) {
    const long long items = (long long)d.zchunks * ((d.n + 4 * kGzRows - 1) / (4 * kGzRows)) * ((d.n + 63) / 64);
    KP_F_SWITCH(k_kp_grad_z, dim3(blocks_of(items)));
    hipLaunchKernelGGL(k_kp_grad_z_sum, dim3(grid_of((long long)d.ns * d.n * d.n * d.F)), dim3(kThreads), 0, s, d);
    return hipGetLastError();
}
// Features FF on the shape that kp_one_bs chooses, `parts` waves a block with two (b, s) a wave.
#define KP_GX(KERNEL, FF, PARTS, ...)                                                                             \
    case FF:                                                                                                      \
        if (kp_one_bs(d)) hipLaunchKernelGGL((KERNEL<FF, 1, kWideParts __VA_OPT__(,) __VA_ARGS__>),               \
                                             dim3(blocks_of(nseg * nbs)), dim3(64 * kWideParts), 0, s, d);        \
        else hipLaunchKernelGGL((KERNEL<FF, (FF > 8 ? 1 : 2), PARTS __VA_OPT__(,) __VA_ARGS__>),                    \
                                dim3(blocks_of(nseg * ((nbs + 1) / 2))), dim3(64 * PARTS), 0, s, d);              \
        break
#define KP_GX_SWITCH(KERNEL, PARTS, ...)                                                                      \
    const long long nseg = (d.n + 63) / 64, nbs = (long long)d.B * d.S;                                       \
    switch (d.F) {                                                                                            \
        KP_GX(KERNEL, 1, PARTS __VA_OPT__(,) __VA_ARGS__); KP_GX(KERNEL, 2, PARTS __VA_OPT__(,) __VA_ARGS__); \
        KP_GX(KERNEL, 4, PARTS __VA_OPT__(,) __VA_ARGS__); KP_GX(KERNEL, 8, PARTS __VA_OPT__(,) __VA_ARGS__); \
        KP_GX(KERNEL, 16, PARTS __VA_OPT__(,) __VA_ARGS__);                                                   \
        default: return hipErrorInvalidValue;                                                                 \
    }                                                                                                         \
    return hipGetLastError()

hipError_t kp_launch_back_x(const KPDesc& d, hipStream_t s) { KP_GX_SWITCH(k_kp_grad_x, kGxParts); }
hipError_t kp_launch_back_y(const KPDesc& d, hipStream_t s) {
    if ((d.n & 1) == 0 && ((uintptr_t)d.G & 15) == 0) { KP_GX_SWITCH(k_kp_grad_y, kGyParts, true); }
    KP_GX_SWITCH(k_kp_grad_y, kGyParts, false);
}
#undef KP_GX_SWITCH
#undef KP_GX
hipError_t kp_launch_back(const KPDesc& d, hipStream_t s) {
    hipError_t e = kp_launch_back_z(d, s);
    if (e == hipSuccess) e = kp_launch_back_x(d, s);
    if (e == hipSuccess) e = kp_launch_back_y(d, s);
    return e;
}
#undef KP_F_SWITCH

hipError_t kp_launch_chain(const KPDesc& d, hipStream_t s) {
    const long long total = 2LL * d.ns * d.S * d.n * d.F + 2LL * d.ns * d.B * d.n * d.F;
    hipLaunchKernelGGL(k_kp_chain1, dim3(grid_of(total)), dim3(kThreads), 0, s, d);
    hipLaunchKernelGGL(k_kp_chain_h, dim3(grid_of((long long)d.ns * d.B * d.S * d.F * 64)), dim3(kThreads), 0, s, d);
    hipLaunchKernelGGL(k_kp_chain_a, dim3(d.F), dim3(kThreads), 0, s, d);
    hipLaunchKernelGGL(k_kp_grid, dim3(grid_of(d.n_params)), dim3(kThreads), 0, s, d);
    return hipGetLastError();
}

hipError_t kp_launch_update(const KPDesc& d, hipStream_t s) {
    hipLaunchKernelGGL(k_kp_update, dim3(grid_of(d.n_params)), dim3(kThreads), 0, s, d);
    if (d.step) hipLaunchKernelGGL(k_kp_advance, dim3(1), dim3(64), 0, s, d.step);
    return hipGetLastError();
}

int kp_reg_blocks(const KPDesc& d) {
    const long long g = (d.a_off + kThreads - 1) / kThreads;
    return (int)(g < 1 ? 1 : (g > 1024 ? 1024 : g));
}

hipError_t kp_launch_reg_value(const KPDesc& d, hipStream_t s) {
    hipLaunchKernelGGL(k_kp_reg_value, dim3(kp_reg_blocks(d)), dim3(kThreads), 0, s, d);
    return hipGetLastError();
}

hipError_t kp_launch_render(const KPDesc& d, int split, float2* proj, float2* water, float2* fat, hipStream_t s) {
    const long long total = (long long)d.B * d.n * d.n;
    KP_IX(k_kp_render, total, d, split, proj, water, fat);
    return hipGetLastError();
}

}  // namespace vp
