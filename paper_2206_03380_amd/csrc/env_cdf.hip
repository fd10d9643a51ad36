// Sampling tables of the lat-long probe (piecewise-constant 2D distribution,
// paper section 4.1 / appendix D), rebuilt whenever the probe changes.
//
// The weights and their running sums are FP64 and summed left to right, the
// order the tables are defined in, so every FP32 entry is the single rounding
// of the same FP64 value on any device.  Three launches:
//   rows      one workgroup per four rows: the lanes compute the weights into
//             LDS, a lane each runs the scans, the lanes write the rows' CDFs
//             and their search guides from LDS;
//   marginal  one workgroup: the scan over the rows' sums;
//   texels    density, packed radiance, density classes and hot slots from one
//             read of the probe.
// What bounds it: the chains of W, then H dependent FP64 adds (12 cycles an
// entry with their LDS accesses: the scan reads 16 entries ahead of its adds),
// and the texels' 36 bytes.  A 1024 x 2048 probe's tables in nine launches
// (a read, an add and a write one after another in the scans, a sine and three
// more reads of the tables per texel) took 119 us of kernels and 133 us a
// build, now 65 and 62.
#include <hip/hip_runtime.h>
#include <math.h>

#include "device_common.h"

#pragma clang fp contract(off)

namespace mcdi {
namespace {

constexpr double kPiD = 3.14159265358979323846;

__device__ __forceinline__ double row_sin(int i, int H) { return sin(kPiD * ((double)i + 0.5) / (double)H); }

__device__ __forceinline__ double texel_weight(const float* env, int W, int i, int j, double srow) {
    const float* t = env + ((size_t)i * W + j) * 3;
    double y = ((double)t[0] + (double)t[1] + (double)t[2]) / 3.0;
    if (!(y > 0.0) || !isfinite(y)) y = 0.0;
    return y * srow;
}

// inclusive prefix of w[0..n) in place, left to right, by one lane; returns
// the sum.  The next 16 entries are read while the present ones are added.
constexpr int kScanAhead = 16;
__device__ __forceinline__ void scan_read(const double* w, double (&v)[kScanAhead]) {
#pragma unroll
    for (int u = 0; u < kScanAhead; ++u) v[u] = w[u];
}
__device__ __forceinline__ void scan_add(double* w, const double (&v)[kScanAhead], double& run) {
#pragma unroll
    for (int u = 0; u < kScanAhead; ++u) {
        run += v[u];
        w[u] = run;
    }
}
__device__ double scan_lane(double* w, int n) {
    constexpr int U = kScanAhead;
    double run = 0.0, a[U], b[U];
    int j = 0;
    if (n >= U) scan_read(w, a);
    for (; j + 3 * U <= n; j += 2 * U) {   // a holds [j, j + U)
        scan_read(w + j + U, b);
        scan_add(w + j, a, run);
        scan_read(w + j + 2 * U, a);
        scan_add(w + j + U, b, run);
    }
    if (j + U <= n) {
        scan_add(w + j, a, run);
        j += U;
    }
    for (; j < n; ++j) {
        run += w[j];
        w[j] = run;
    }
    return run;
}

// Rows a workgroup builds: their scans run on neighbouring lanes of one
// wavefront.  An LDS access of one lane takes the LDS as long as one of
// several, and with one row per workgroup the scans of the workgroups on a CU
// shared its LDS: 61 cycles per entry against 12 for a lone scan (2048 columns).
constexpr int kRowsPer = 4;
constexpr int kRowThreads = 1024;
inline int rows_per_group(int W) { return W > 2048 ? 2 : kRowsPer; }   // 64 KB of LDS and the padding
// doubles of LDS a row takes: the scanning lanes' rows start 16 bytes apart
// modulo the banks
__host__ __device__ constexpr int row_stride(int W) { return W + 2; }

// rowsum: [H] row sums, [H] the total (marginal_kernel), [H + 1 ..) the rows' sines
__global__ __launch_bounds__(kRowThreads) void rows_kernel(const float* env, int H, int W, int G, int rows, float* cond,
                                                           double* rowsum, uint16_t* guide, int32_t* n_hot) {
    extern __shared__ double smem[];  // [rows][row_stride(W)]
    __shared__ double s_sum[kRowsPer], s_sin[kRowsPer];
    const int i0 = blockIdx.x * rows, nr = min(rows, H - i0), S = row_stride(W);
    if (threadIdx.x < nr) s_sin[threadIdx.x] = row_sin(i0 + threadIdx.x, H);
    __syncthreads();
    for (int r = 0; r < nr; ++r)
        for (int j = threadIdx.x; j < W; j += kRowThreads) smem[r * S + j] = texel_weight(env, W, i0 + r, j, s_sin[r]);
    __syncthreads();
    if (threadIdx.x < nr) {
        const int r = threadIdx.x;
        s_sum[r] = scan_lane(smem + r * S, W);
        rowsum[i0 + r] = s_sum[r];
        rowsum[H + 1 + i0 + r] = s_sin[r];
        if (i0 + r == 0) *n_hot = 0;
    }
    __syncthreads();
    // entry k >= 1 replaces the prefix it is made of (slot k - 1, its own lane's)
    auto entry = [&](int r, int k) -> float& { return *reinterpret_cast<float*>(smem + r * S + (k - 1)); };
    for (int r = 0; r < nr; ++r) {
        const double rs = s_sum[r];
        float* c = cond + (size_t)(i0 + r) * (W + 1);
        for (int k = threadIdx.x; k <= W; k += kRowThreads) {
            float v;
            if (k == 0) v = 0.0f;
            else if (k == W) v = 1.0f;
            else v = rs > 0.0 ? (float)(smem[r * S + k - 1] / rs) : (float)((double)k / (double)W);
            if (k > 0) entry(r, k) = v;
            c[k] = v;
        }
    }
    __syncthreads();
    // guide[g] = the largest column k <= W - 1 with cond[k] <= g / G
    for (int q = threadIdx.x; q < nr * (G + 1); q += kRowThreads) {
        const int r = q / (G + 1), g = q - r * (G + 1);
        const float x = (float)g / (float)G;
        int lo = 0, hi = W;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (entry(r, mid) <= x) lo = mid; else hi = mid;
        }
        guide[(size_t)(i0 + r) * (G + 1) + g] = (uint16_t)lo;
    }
}

__global__ __launch_bounds__(256) void marginal_kernel(const double* rowsum, int H, float* marg, double* total_out,
                                                        int32_t* light_enabled) {
    extern __shared__ double pre[];  // [H]
    __shared__ double s_tot;
    for (int k = threadIdx.x; k < H; k += blockDim.x) pre[k] = rowsum[k];
    __syncthreads();
    if (threadIdx.x == 0) {
        const double run = scan_lane(pre, H);
        s_tot = run;
        *total_out = run;
        *light_enabled = run > 0.0 ? 1 : 0;
    }
    __syncthreads();
    const double tot = s_tot;
    for (int k = threadIdx.x; k <= H; k += blockDim.x) {
        float v;
        if (k == 0) v = 0.0f;
        else if (k == H) v = 1.0f;
        else v = tot > 0.0 ? (float)(pre[k - 1] / tot) : (float)((double)k / (double)H);
        marg[k] = v;
    }
}

// Per texel:
//  pdf     its density in (u, v);
//  tex     (r, g, b, pdf);
//  dclass  two bits for ray generation, which only asks whether a light sample
//          has a density: 0 none (pdf <= 0 or NaN: pdf / (2 pi^2 sin) is not
//          > 0), 1 pdf >= 2^-100 (then pdf / (2 pi^2 sin) > 0 for every sin in
//          (0, 1]: the quotient is at least 2^-100 / 19.8, or infinite), 2 a
//          tiny positive pdf, whose quotient may round to 0 (read the pdf).  A
//          quarter of a byte per texel stays in the L2 cache where the 4-byte
//          densities do not;
//  hot     texels the light technique samples with probability above
//          1/kHotMax get a slot (at most kHotMax of them, since the
//          probabilities sum to 1): the adjoint accumulates their gradient per
//          workgroup in LDS before one global atomic per slot and workgroup.
// Four neighbouring lanes share a byte of classes.
__global__ __launch_bounds__(256) void texel_kernel(const float* __restrict__ env, int H, int W,
                                                    const double* __restrict__ rowsum, float* __restrict__ pdf,
                                                    float4* __restrict__ tex, uint8_t* __restrict__ dclass,
                                                    int32_t* __restrict__ hot_slot, int32_t* __restrict__ hot_texel,
                                                    int32_t* n_hot) {
    const int n = H * W;
    const int k = (int)(blockIdx.x * 256 + threadIdx.x);
    uint32_t cls = 0;
    if (k < n) {
        const int i = k / W, j = k - i * W;
        const double tot = rowsum[H];
        const double w = texel_weight(env, W, i, j, rowsum[H + 1 + i]);
        const float p = tot > 0.0 ? (float)((w / tot) * ((double)W * (double)H)) : 0.0f;
        const float* c = env + 3 * (size_t)k;
        pdf[k] = p;
        tex[k] = make_float4(c[0], c[1], c[2], p);
        cls = !(p > 0.0f) ? 0u : (p >= 0x1p-100f ? 1u : 2u);
        int32_t slot = -1;
        if (p / ((float)W * (float)H) > 1.0f / (float)kHotMax) {
            slot = atomicAdd(n_hot, 1);
            if (slot < kHotMax) hot_texel[slot] = k;
            else slot = -1;
        }
        hot_slot[k] = slot;
    }
    cls <<= 2 * (threadIdx.x & 3);
    cls |= __shfl_xor(cls, 1);
    cls |= __shfl_xor(cls, 2);
    if (k < n && (threadIdx.x & 3) == 0) dclass[k >> 2] = (uint8_t)cls;
}

__global__ __launch_bounds__(256) void mix_kernel(const float4* rgb, const float4* dens, int64_t n, float4* out) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const float4 a = rgb[k];
    out[k] = make_float4(a.x, a.y, a.z, dens[k].w);
}

}  // namespace

hipError_t launch_env_mix(const float4* rgb, const float4* dens, int64_t n, float4* out, hipStream_t s) {
    hipLaunchKernelGGL(mix_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, rgb, dens, n, out);
    return hipGetLastError();
}

// Guide cells per row, at most 1024: about eight columns per cell, sixteen where
// the conditional table is larger than one XCD's L2 (4 MB): draws wait for its
// lines there, and a guide of half the size leaves them more of the cache.
// Generation and forward shading of 4.2M pixels at 32 spp, 4, 8, 16 and 32
// columns: 512 x 1024 probe 3.43, 3.31, 3.45 ms (4, 8, 16), 1024 x 2048 probe
// 4.83, 4.37, 4.34, 4.72 ms.
int env_guide_cells(int H, int W) {
    constexpr double kL2Bytes = 4 << 20;
    const int cols = (double)H * (W + 1) * sizeof(float) > kL2Bytes ? 16 : 8;
    int G = 1;
    while (cols * G <= W && G < 1024) G *= 2;
    return G;
}

hipError_t launch_env_tables(const float* env, int H, int W, const EnvTables& t, hipStream_t s) {
    const int rows = rows_per_group(W);
    const size_t lds = sizeof(double) * (size_t)rows * (size_t)row_stride(W);
    if (lds > 65536) {   // above the default dynamic LDS limit (by the rows' padding)
        const hipError_t e = hipFuncSetAttribute((const void*)rows_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(rows_kernel, dim3((unsigned)((H + rows - 1) / rows)), dim3(kRowThreads), lds, s, env, H, W, t.G,
                       rows, t.cond, t.rowsum, t.guide, t.n_hot);
    hipLaunchKernelGGL(marginal_kernel, dim3(1), dim3(256), sizeof(double) * (size_t)H, s, t.rowsum, H, t.marg,
                       t.rowsum + H, t.light_enabled);
    const int64_t n = (int64_t)H * W;
    hipLaunchKernelGGL(texel_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, env, H, W, t.rowsum, t.pdf,
                       t.tex, t.dclass, t.hot_slot, t.hot_texel, t.n_hot);
    return hipGetLastError();
}

}  // namespace mcdi
