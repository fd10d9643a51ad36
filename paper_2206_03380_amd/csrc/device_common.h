// Device building blocks for gfx950: counter-based RNG, probe sampling, GGX
// material model, visible-normal sampling and the any-hit BVH traversal.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mcdi_internal.h"

namespace mcdi {

constexpr float kPi = 3.14159265358979323846f;
constexpr float kInvPi = 0.318309886183790671538f;
constexpr float kRMin = 0.08f;  // roughness clamp (alpha >= 0.0064)
// Word 3 of a raw buffer resource on gfx9 (data format 32, no swizzle): the
// descriptor of __builtin_amdgcn_make_buffer_rsrc for plain byte-offset loads.
constexpr int kBufferWord3 = 0x00020000;
constexpr uint32_t kNone = 0xFFFFFFFFu;

// decision-record bits (debug dump)
constexpr uint32_t kDecLobeCos = 1u << 0, kDecLCull = 1u << 1, kDecBCull = 1u << 2;
constexpr uint32_t kDecLTraced = 1u << 3, kDecBTraced = 1u << 4, kDecLHit = 1u << 5;
constexpr uint32_t kDecBHit = 1u << 6, kDecNovPos = 1u << 7, kDecValid = 1u << 8;

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC 2011): ten rounds of two 32x32 products.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint4 philox10(uint4 c, uint32_t k0, uint32_t k1) {
    // each 32 x 32 -> 64-bit product as one multiply (both halves at once)
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c.x, p1 = (uint64_t)0xCD9E8D57u * c.z;
        c = make_uint4(xor3((uint32_t)(p1 >> 32), c.y, k0), (uint32_t)p1, xor3((uint32_t)(p0 >> 32), c.w, k1), (uint32_t)p0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// top 24 bits as a float in [0, 1), exact
__device__ __forceinline__ float u01(uint32_t x) { return (float)(x >> 8) * 0x1p-24f; }

// ---------------------------------------------------------------------------
// small vector helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ float3 f3(float x, float y, float z) { return make_float3(x, y, z); }
__device__ __forceinline__ float dot(float3 a, float3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ float3 operator+(float3 a, float3 b) { return f3(a.x + b.x, a.y + b.y, a.z + b.z); }
__device__ __forceinline__ float3 operator-(float3 a, float3 b) { return f3(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ __forceinline__ float3 operator*(float s, float3 a) { return f3(s * a.x, s * a.y, s * a.z); }
__device__ __forceinline__ float3 normalize(float3 a) { return (1.0f / sqrtf(dot(a, a))) * a; }

// ---------------------------------------------------------------------------
// CDF searches: the largest k in [0, n-1] with cdf[k] <= x (cdf[0] = 0 <= x <
// 1 = cdf[n], non-decreasing) -- skips zero-width bins.
// ---------------------------------------------------------------------------
// Binary search without bounds: the table is padded to search_size(n) entries
// above x (as entry n is), so each halving is one read, one compare and one
// select at addresses that need no check.
__host__ __device__ inline int search_size(int n) {
    return n > 1 ? 1 << (32 - __builtin_clz((unsigned)(n - 1))) : 1;
}
__device__ __forceinline__ int cdf_find_padded(const float* cdf, int size, float x) {
    int k = 0;
    for (int step = size >> 1; step > 0; step >>= 1) k = cdf[k + step] <= x ? k + step : k;
    return k;
}

// a / b for b = 1..4096 by its correctly rounded reciprocal rb: the quotient of
// the rounded product is corrected by its exact remainder (Markstein 1990).
// The result is the correctly rounded quotient for every such b and every a
// whose remainder does not underflow (all 2^23 significands of a tried for each
// b), at three instructions instead of the ten of a division.
__device__ __forceinline__ float div_small(float a, float b, float rb) {
    const float q = a * rb;
    return fmaf(fmaf(-q, b, a), rb, q);
}

// columns [lo, hi) that a guide cell's draws can fall into (two neighbouring
// entries in one load)
__device__ __forceinline__ void guide_cell(const uint16_t* guide, int& lo, int& hi) {
    uint32_t two;
    __builtin_memcpy(&two, guide, 4);
    lo = (int)(two & 0xFFFFu);
    hi = (int)(two >> 16) + 1;
}

// The same search with the row's guide (guide[g] = the answer for g / G,
// g = 0..G, G a power of two): for x in [0, 1) with g = floor(x G), the
// answer lies in [guide[g], guide[g + 1]], since g / G <= x < (g + 1) / G and
// both bounds are exact in FP32; the binary search over that range returns
// the same column as one over the whole row.
__device__ __forceinline__ int cdf_find_guided(const float* cdf, const uint16_t* guide, int G, float x) {
    const int g = min(max((int)(x * (float)G), 0), G - 1);
    int lo, hi;
    guide_cell(guide + g, lo, hi);
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cdf[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// The guided search of one conditional row with the candidates read in one
// go, and the CDF values on both sides of the answer (c0 = cdf[j],
// c1 = cdf[j + 1]).  Four aligned 16-byte loads, issued together, cover the
// 13 to 16 entries from the cell's first candidate on.  Over a non-decreasing
// CDF the answer is the first candidate plus the number of later candidates
// (below the cell's end) that are <= x; if every candidate in the window is,
// the binary search goes on behind them.  One round trip for the candidates
// instead of one per probe: with many waves in flight a line read by one probe
// is often evicted before the next (cdf_find_guided's probes then each go to
// memory).  The row must be 4-byte aligned within a 16-byte aligned table that
// extends at least 16 floats past the row's last entry.
//
// Candidates are counted in one bit mask (two instructions each; a compare
// against the cell's bounds per candidate took four and spilled scalar
// registers), and the two values come from the registers by a tree of selects
// (reading them again cost more than the search saves: the lines are gone).
// Generation and forward shading of 4.2M pixels at 32 spp, before (window only
// for tables past 4 MB) -> now, with the draws' other instructions: probes of
// 64, 256, 512, 1024 and 1500 rows 3.05 -> 2.76, 3.76 -> 3.08, 4.03 -> 3.31,
// 4.65 -> 4.34, 5.71 -> 5.02 ms.
__device__ __forceinline__ int cdf_find_row(const float* cdf, const uint16_t* guide, int G, float x, float& c0,
                                            float& c1) {
    constexpr int NW = 16;
    const int g = min(max((int)(x * (float)G), 0), G - 1);
    int lo, hi;
    guide_cell(guide + g, lo, hi);
    const float* p = cdf + lo;
    const int o = (int)(((uintptr_t)p >> 2) & 3u);
    const float4* a = (const float4*)(p - o);
    float4 w0 = a[0], w1 = a[1], w2 = a[2], w3 = a[3];
    // (opaque from here on: kept as four aligned loads, and as registers)
    asm("" : "+v"(w0.x), "+v"(w0.y), "+v"(w0.z), "+v"(w0.w), "+v"(w1.x), "+v"(w1.y), "+v"(w1.z), "+v"(w1.w));
    asm("" : "+v"(w2.x), "+v"(w2.y), "+v"(w2.z), "+v"(w2.w), "+v"(w3.x), "+v"(w3.y), "+v"(w3.z), "+v"(w3.w));
    // window slot t holds cdf[lo - o + t]; bit t of gt tells whether it is > x,
    // by the difference of the patterns (neither is negative)
    const uint32_t xb = __float_as_uint(x);
    uint32_t gt = 0u;
    auto push = [&](float v) { gt = __builtin_amdgcn_alignbit(gt, xb - __float_as_uint(v), 31u); };
    push(w3.w); push(w3.z); push(w3.y); push(w3.x);
    push(w2.w); push(w2.z); push(w2.y); push(w2.x);
    push(w1.w); push(w1.z); push(w1.y); push(w1.x);
    push(w0.w); push(w0.z); push(w0.y); push(w0.x);
    // later candidates in the window (slots o + 1 .. o + span - 1) that are <= x
    const uint32_t in = ((2u << min(hi - lo - 1, NW - 1)) - 2u) << o;
    const int cnt = __popc(~gt & in & ((1u << NW) - 1u));
    lo += cnt;
    if (cnt < NW - 1 - o) {
        // slots s and s + 1 of the window by the bits of s
        const int s = o + cnt;
        const bool s1 = (s & 1) != 0, s2 = (s & 2) != 0, s4 = (s & 4) != 0, s8 = (s & 8) != 0;
        const float a0 = s1 ? w0.y : w0.x, a1 = s1 ? w0.w : w0.z, a2 = s1 ? w1.y : w1.x, a3 = s1 ? w1.w : w1.z;
        const float a4 = s1 ? w2.y : w2.x, a5 = s1 ? w2.w : w2.z, a6 = s1 ? w3.y : w3.x, a7 = s1 ? w3.w : w3.z;
        const float b0 = s1 ? w0.z : w0.y, b1 = s1 ? w1.x : w0.w, b2 = s1 ? w1.z : w1.y, b3 = s1 ? w2.x : w1.w;
        const float b4 = s1 ? w2.z : w2.y, b5 = s1 ? w3.x : w2.w, b6 = s1 ? w3.z : w3.y, b7 = w3.w;
        const float c00 = s2 ? a1 : a0, c01 = s2 ? a3 : a2, c02 = s2 ? a5 : a4, c03 = s2 ? a7 : a6;
        const float d00 = s2 ? b1 : b0, d01 = s2 ? b3 : b2, d02 = s2 ? b5 : b4, d03 = s2 ? b7 : b6;
        const float e0 = s4 ? c01 : c00, e1 = s4 ? c03 : c02, f0 = s4 ? d01 : d00, f1 = s4 ? d03 : d02;
        c0 = s8 ? e1 : e0;
        c1 = s8 ? f1 : f0;
        return lo;
    }
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cdf[mid] <= x) lo = mid; else hi = mid;
    }
    c0 = cdf[lo];
    c1 = cdf[lo + 1];
    return lo;
}

// ---------------------------------------------------------------------------
// GGX with Smith height-correlated masking (alpha = roughness^2)
// ---------------------------------------------------------------------------
// D written with s2 = |n x h|^2 (local: h.x^2 + h.y^2) for 1 - (n.h)^2
__device__ __forceinline__ float ggx_D(float noh, float s2, float a2) {
    const float den = a2 * noh * noh + s2;
    return a2 / (kPi * den * den);
}

__device__ __forceinline__ float smith_t2(float x) { return (1.0f - x * x) / (x * x); }

__device__ __forceinline__ float smith_lambda(float t2, float a2) {
    return 0.5f * (sqrtf(1.0f + a2 * t2) - 1.0f);
}

// ---------------------------------------------------------------------------
// Watertight ray/triangle test (Woop, Benthin, Wald; JCGT 2013), any hit with
// t in (0, inf).  The ray is pre-sheared: kz is the dominant axis of d, and a
// vertex's sheared coordinates are (v - o)[kx] - sx (v - o)[kz] and
// (v - o)[ky] - sy (v - o)[kz].  Edge functions use no contraction so a
// shared edge gives exactly negated values in its two triangles; an
// exactly-zero edge function is re-evaluated in FP64.
//
// A triangle is stored by axis: three rows (v0, v1, v2, 0) of its x, y and z
// coordinates, so a ray reads the rows kx, ky and kz (three 16-byte loads at
// its own offsets) and the test neither selects components nor multiplies by
// a shear matrix's zeros and ones: about
// 50 instructions against 80.  Shadow rays of a room of 1.0M triangles 9.6 ->
// 8.8 ms, of a 102k-triangle surface 2.26 -> 2.12 ms.
//
// Rays that graze an edge are decided by the last bit of the sheared
// coordinates, so their rounding is part of the answer: row . (v - o) is
// summed over x, y, z with y's product rounded and the other two fused.  A row
// holds a one, a zero and -s (at kz), so the sum has one rounding where kz = z
// and on the row of y where kz = x, and elsewhere two (the product's first).
// A ray's (c, e) = (-s, 1) or (-1, s) gives either by one multiply and one FMA,
// c (e z) + x: the product with a one is exact.
//
// Loads go by 32-bit byte offsets from the first triangle (below 2^26 triangles
// of 48 bytes): 64-bit addresses cost two registers and spilled the walk.
//
// kx and ky stay in cyclic order when d[kz] < 0 (the published test swaps
// them to keep the winding): the swap negates U, V, W, their sum and T exactly,
// and a hit from either side counts.
// ---------------------------------------------------------------------------
struct Ray {
    float3 o;
    float3 inv;      // 1/d (zero components replaced, boxes only)
    float3 clo, chi; // slab offsets for the low and high box corners (box_hit)
    float3 p;        // o[kx], o[ky], o[kz]
    float cx, ex;    // shear of row kx, s = d[kx] / d[kz]: (-s, 1) where s z is fused into the sum, (-1, s) where rounded
    float cy, ey;    // the same of row ky
    float sz;        // 1/d[kz]
    uint32_t rx, ry, rz;   // byte offsets of the rows kx, ky, kz
};

// Slab offsets: t = corner * inv + c with c = -(o * inv) -/+ e on the near/far
// side of each axis.  o*inv is rounded once, so e = 2^-21 |o*inv| (eight times
// that rounding plus the rounding of c itself) keeps every near distance an
// under- and every far distance an over-estimate before the final rounding of
// the FMA.
__device__ __forceinline__ void slab_offsets(float o, float inv, float& clo, float& chi) {
    const float oi = o * inv;
    const float e = fabsf(oi) * 0x1p-21f;
    const float cn = -oi - e, cf = -oi + e;
    clo = inv >= 0.0f ? cn : cf;
    chi = inv >= 0.0f ? cf : cn;
}

__device__ __forceinline__ float comp(float3 v, int k) { return k == 0 ? v.x : (k == 1 ? v.y : v.z); }

// Reciprocals use the hardware approximation (<= 1 ulp): the shear constants
// only need to be the same for every triangle a ray meets, and the box test
// widens t_far for the extra ulp.
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

__device__ __forceinline__ Ray make_ray(float3 o, float3 d) {
    Ray r;
    r.o = o;
    const float ax = fabsf(d.x), ay = fabsf(d.y), az = fabsf(d.z);
    const int kz = (ax > ay) ? (ax > az ? 0 : 2) : (ay > az ? 1 : 2);
    const int kx = kz == 2 ? 0 : kz + 1;
    const int ky = kx == 2 ? 0 : kx + 1;
    const float rz = fast_rcp(comp(d, kz));
    r.p = f3(comp(o, kx), comp(o, ky), comp(o, kz));
    const float sx = comp(d, kx) * rz, sy = comp(d, ky) * rz;
    const bool fx = kz != 1, fy = kz == 2;   // row kx = y at kz = x; both at kz = z
    r.cx = fx ? -sx : -1.0f;
    r.ex = fx ? 1.0f : sx;
    r.cy = fy ? -sy : -1.0f;
    r.ey = fy ? 1.0f : sy;
    r.sz = rz;
    r.rx = 16u * (uint32_t)kx;
    r.ry = 16u * (uint32_t)ky;
    r.rz = 16u * (uint32_t)kz;
    const float tiny = 1e-30f;
    r.inv = f3(fast_rcp(d.x != 0.0f ? d.x : tiny), fast_rcp(d.y != 0.0f ? d.y : tiny),
               fast_rcp(d.z != 0.0f ? d.z : tiny));
    slab_offsets(o.x, r.inv.x, r.clo.x, r.chi.x);
    slab_offsets(o.y, r.inv.y, r.clo.y, r.chi.y);
    slab_offsets(o.z, r.inv.z, r.clo.z, r.chi.z);
    return r;
}

__device__ __forceinline__ bool tri_anyhit(const Ray& r, const void* tris, uint32_t at) {
#pragma clang fp contract(off)
    const char* t = static_cast<const char*>(tris);
    const float4 vx = *reinterpret_cast<const float4*>(t + (at + r.rx));
    const float4 vy = *reinterpret_cast<const float4*>(t + (at + r.ry));
    const float4 vz = *reinterpret_cast<const float4*>(t + (at + r.rz));
    const float az = vz.x - r.p.z, bz = vz.y - r.p.z, cz = vz.z - r.p.z;
    const float Ax = fmaf(r.cx, r.ex * az, vx.x - r.p.x), Ay = fmaf(r.cy, r.ey * az, vy.x - r.p.y);
    const float Bx = fmaf(r.cx, r.ex * bz, vx.y - r.p.x), By = fmaf(r.cy, r.ey * bz, vy.y - r.p.y);
    const float Cx = fmaf(r.cx, r.ex * cz, vx.z - r.p.x), Cy = fmaf(r.cy, r.ey * cz, vy.z - r.p.y);
    float U = Cx * By - Cy * Bx;
    float V = Ax * Cy - Ay * Cx;
    float W = Bx * Ay - By * Ax;
    if (U == 0.0f || V == 0.0f || W == 0.0f) {
        U = (float)((double)Cx * (double)By - (double)Cy * (double)Bx);
        V = (float)((double)Ax * (double)Cy - (double)Ay * (double)Cx);
        W = (float)((double)Bx * (double)Ay - (double)By * (double)Ax);
    }
    if ((U < 0.0f || V < 0.0f || W < 0.0f) && (U > 0.0f || V > 0.0f || W > 0.0f)) return false;
    const float det = U + V + W;
    if (det == 0.0f) return false;
    const float T = U * (r.sz * az) + V * (r.sz * bz) + W * (r.sz * cz);
    return det > 0.0f ? (T > 0.0f) : (T < 0.0f);
}

// Conservative slab test (Ize 2013: widen t_far by 1 + 2 gamma(n)), t >= 0;
// n = 4 covers the subtraction, the product and the 1-ulp reciprocal, and the
// factor is rounded up.
__device__ __forceinline__ bool box_hit(const Ray& r, float4 a, float4 b) {
    const float tx0 = fmaf(a.x, r.inv.x, r.clo.x), tx1 = fmaf(b.x, r.inv.x, r.chi.x);
    const float ty0 = fmaf(a.y, r.inv.y, r.clo.y), ty1 = fmaf(b.y, r.inv.y, r.chi.y);
    const float tz0 = fmaf(a.z, r.inv.z, r.clo.z), tz1 = fmaf(b.z, r.inv.z, r.chi.z);
    const float tn = fmaxf(fmaxf(fminf(tx0, tx1), fminf(ty0, ty1)), fmaxf(fminf(tz0, tz1), 0.0f));
    const float tf = fminf(fminf(fmaxf(tx0, tx1), fmaxf(ty0, ty1)), fmaxf(tz0, tz1));
    return tn <= tf * 1.000001f;
}

// Slab constants of a ray against the scene's quantisation frame: the plane v
// of axis a lies at mid + v step, so t = v (step inv) + (mid - o) inv, one
// mixed-precision FMA per plane that reads the half-precision coordinate
// straight from its half of the word (v_fma_mix_f32: no conversion).  The
// offsets carry a margin of 2^-20 (65535 |step inv| + |(mid - o) inv|), |v|
// being at most 2^15 (65504 in an empty record) -- sixteen times the roundings
// of the two products, the difference and the FMA against the magnitudes
// involved -- on the side that keeps near distances under- and far distances
// over-estimated; they also cover the reciprocal's 1-ulp error, so the final
// comparison needs no slack.
// Which plane of an axis is near follows from the sign of the direction: per
// axis a byte selector gathers the near plane's coordinate (low half) and the
// far plane's (high half) from the two words holding them, so that the test
// needs no min/max pairs.
// 13 instructions a box: 3 permutes, 6 FMAs, 3 min/max and a compare.  With
// 16-bit integer coordinates six conversions came on top (shadow rays of a
// surface: 1.45e9 -> 1.27e9 vector instructions a launch).
struct QRay {
    float3 s, cn, cf;
    uint32_t sx, sy, sz;
};

__device__ __forceinline__ void qslab(float o, float inv, float mid, float step, float& s, float& cn,
                                      float& cf) {
    s = step * inv;
    const float c = (mid - o) * inv;
    const float e = 0x1p-20f * (fabsf(s) * 65535.0f + fabsf(c));
    cn = c - e;
    cf = c + e;
}

__device__ __forceinline__ QRay make_qray(const Ray& r, const QFrame& F) {
    QRay q;
    qslab(r.o.x, r.inv.x, F.mid[0], F.step[0], q.s.x, q.cn.x, q.cf.x);
    qslab(r.o.y, r.inv.y, F.mid[1], F.step[1], q.s.y, q.cn.y, q.cf.y);
    qslab(r.o.z, r.inv.z, F.mid[2], F.step[2], q.s.z, q.cn.z, q.cf.z);
    // x: lo in word 0 of n.x, hi in word 1 of n.y; y: lo in word 1 of n.x,
    // hi in word 0 of n.z; z: lo in word 0 of n.y, hi in word 1 of n.z
    // (selector bytes 0-3 take the second operand, 4-7 the first)
    q.sx = r.inv.x >= 0.0f ? 0x07060100u : 0x01000706u;
    q.sy = r.inv.y >= 0.0f ? 0x05040302u : 0x03020504u;
    q.sz = r.inv.z >= 0.0f ? 0x07060100u : 0x01000706u;
    return q;
}

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ bool qbox_hit(const QRay& q, uint4 n) {
    const half2_t ax = __builtin_bit_cast(half2_t, __builtin_amdgcn_perm(n.y, n.x, q.sx));
    const half2_t ay = __builtin_bit_cast(half2_t, __builtin_amdgcn_perm(n.z, n.x, q.sy));
    const half2_t az = __builtin_bit_cast(half2_t, __builtin_amdgcn_perm(n.z, n.y, q.sz));
    const float tnx = fmaf((float)ax.x, q.s.x, q.cn.x), tfx = fmaf((float)ax.y, q.s.x, q.cf.x);
    const float tny = fmaf((float)ay.x, q.s.y, q.cn.y), tfy = fmaf((float)ay.y, q.s.y, q.cf.y);
    const float tnz = fmaf((float)az.x, q.s.z, q.cn.z), tfz = fmaf((float)az.y, q.s.z, q.cf.z);
    const float tn = fmaxf(fmaxf(fmaxf(tnx, tny), tnz), 0.0f);
    const float tf = fminf(fminf(tfx, tfy), tfz);
    return tn <= tf;
}

// a leaf's triangles (its reference)
template <bool COUNT>
__device__ __forceinline__ bool leaf_anyhit(const Scene& sc, const Ray& r, uint32_t ref, uint32_t& n_tri) {
    const uint32_t first = (ref >> 2) & 0x03FFFFFFu, cnt = (ref & 3u) + 1u;
    for (uint32_t k = first; k < first + cnt && k < (uint32_t)sc.n_tris; ++k) {
        if (COUNT) ++n_tri;
        if (tri_anyhit(r, sc.tris, 48u * k)) return true;
    }
    return false;
}

// octant of a ray: bit a set where the direction is negative on axis a, and
// bit 3, the "axis" of the split that separates the big triangles
__device__ __forceinline__ uint32_t ray_octant(float3 d) {
    return 8u | (d.x < 0.0f ? 1u : 0u) | (d.y < 0.0f ? 2u : 0u) | (d.z < 0.0f ? 4u : 0u);
}
// whether a ray of octant oct takes the split's first child after its second
// in slot order (the last pushed is popped first): the split's axis in a
// record's word
__device__ __forceinline__ bool split_swaps(uint32_t oct, uint32_t word) {
    return ((oct >> ((word >> kRefAxisShift) & 3u)) & 1u) != 0u;
}

// Stackless any-hit traversal over the quantised nodes (the order and the
// skip links of the pre-order BVH; a leaf's escape is the next node).
template <bool COUNT = false>
__device__ __forceinline__ bool qbvh_anyhit(const Scene& sc, const Ray& r, const QRay& q, int n_total,
                                            uint32_t& n_box, uint32_t& n_tri) {
    const uint4* nodes = reinterpret_cast<const uint4*>(sc.qnodes);
    int i = 0;
    while (i < n_total) {
        const uint4 n = nodes[i];
        const bool leaf = (n.w & kQLeaf) != 0u;
        // skip links always point forward; anything else ends the walk
        const int next = leaf ? i + 1 : ((int)n.w > i ? (int)n.w : n_total);
        if (COUNT) ++n_box;
        if (!qbox_hit(q, n)) { i = next; continue; }
        if (!leaf) { ++i; continue; }
        if (leaf_anyhit<COUNT>(sc, r, n.w, n_tri)) return true;
        i = next;
    }
    return false;
}

// Any-hit traversal of the 4-wide hierarchy with a stack of pending
// references (a one-ray form; the shading kernels keep their stacks in LDS).
// Hit children are pushed in the node's visit order for the ray's octant and
// the last pushed is taken next, so each split's farther child comes first,
// as in the shading kernels' walk.  A stack that would overflow sends the ray
// to the binary traversal from the root, which gives the same answer.
template <bool COUNT = false>
__device__ __forceinline__ bool wbvh_anyhit(const Scene& sc, const Ray& r, int n_total, uint32_t& n_box,
                                            uint32_t& n_tri) {
    constexpr int kDepth = 64;
    const uint4* g = reinterpret_cast<const uint4*>(sc.groups);
    const uint32_t n_groups = sc.group_bytes / 64u;
    const QRay q = make_qray(r, *sc.frame);
    const uint32_t oct = ray_octant(r.inv);
    uint32_t stack[kDepth];
    int sp = 0;
    uint32_t node = n_total > 0 ? 0u : kWideNone;
    while (true) {
        if (node == kWideNone) {
            if (sp == 0) return false;
            node = stack[--sp];
        }
        if (node & kQLeaf) {
            if (leaf_anyhit<COUNT>(sc, r, node, n_tri)) return true;
            node = kWideNone;
            continue;
        }
        if (node >= n_groups) { node = kWideNone; continue; }   // never for a valid hierarchy
        const uint4* gn = g + 4 * (size_t)node;
        const bool s0 = split_swaps(oct, gn[1].w), s1 = split_swaps(oct, gn[2].w), sT = split_swaps(oct, gn[0].w);
        // slot order: swap within the first pair, within the second, the pairs
        for (int p = 0; p < 4; ++p) {
            int k = p;
            if (sT) k ^= 2;
            if ((k < 2 && s0) || (k >= 2 && s1)) k ^= 1;
            const uint4 c = gn[k];
            const uint32_t ref = c.w & kRefMask;
            if (COUNT && ref != kEmptyRef) ++n_box;
            if (!qbox_hit(q, c)) continue;
            if (sp >= kDepth) return qbvh_anyhit<COUNT>(sc, r, q, n_total, n_box, n_tri);
            stack[sp++] = ref;
        }
        node = kWideNone;   // the last pushed is popped next
    }
}

// Stackless any-hit traversal over the pre-order BVH with skip links.
// COUNT: tally box tests and triangle tests (statistics instantiation only).
template <bool COUNT = false>
__device__ __forceinline__ bool bvh_anyhit(const Scene& sc, const Ray& r, int n_total, uint32_t& n_box,
                                           uint32_t& n_tri) {
    const float4* nodes = reinterpret_cast<const float4*>(sc.nodes);
    int i = 0;
    while (i < n_total) {
        const float4 a = nodes[2 * i];
        const float4 b = nodes[2 * i + 1];
        const int escape = __float_as_int(a.w);
        const int payload = __float_as_int(b.w);
        // skip links always point forward; anything else ends the walk
        const int next = escape > i ? escape : n_total;
        if (COUNT) ++n_box;
        if (!box_hit(r, a, b)) { i = next; continue; }
        if (payload == 0) { ++i; continue; }
        const int first = payload >> 3;
        const int cnt = (first + (payload & 7) <= sc.n_tris) ? (payload & 7) : 0;
        for (int k = 0; k < cnt; ++k) {
            if (COUNT) ++n_tri;
            if (tri_anyhit(r, sc.tris, 48u * (uint32_t)(first + k))) return true;
        }
        i = next;
    }
    return false;
}

// set bits of m below the lane's own
__device__ __forceinline__ int bits_below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// orders a wavefront's LDS accesses before it against those behind it, of all its
// lanes among each other (no instruction: the LDS serves a wave in order; the
// barrier alone only keeps the compiler from moving what has side effects)
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Any-hit query of one ray by a whole wavefront over the 4-wide hierarchy.  The
// wave keeps one stack of references in LDS: each step takes the top 64 (or
// all), a lane to each -- a node's hit children go back onto the stack, a
// leaf's triangles are tested -- so a ray that misses costs about as many
// dependent steps as the tree has levels, and one that hits stops with the
// step that finds it.  (One lane per subtree, each walking its own with skip
// links, took the longest subtree's walk: 3,400 rays against 102k triangles
// 184 us, now 42.)  A stack that would
// overflow hands the ray to the binary walk of a lane.  The ray must be
// the same in every lane; the result is uniform.
// Entry i of the stack is at [(i / 64) * STRIDE + i % 64].
constexpr int kWaveStack = 1024;
template <int STRIDE, int CAP>
__device__ __forceinline__ bool wave_anyhit(const Scene& sc, const Ray& r, const QRay& q, int n_total,
                                            uint32_t* stack) {
    auto entry = [&](int i) -> uint32_t& { return stack[(i >> 6) * STRIDE + (i & 63)]; };
    if (n_total <= 0) return false;
    const uint4* g = reinterpret_cast<const uint4*>(sc.groups);
    const uint32_t n_groups = sc.group_bytes / 64u;
    const int lane = __lane_id();
    bool flat = sc.info->wide_bad != 0;
    int n = 1;
    if (lane == 0) entry(0) = 0u;
    while (n > 0 && !flat) {
        const int take = min(min(n, 64), max((CAP - n) / 3, 1));   // each gives back four at most
        n -= take;
        bool hit = false;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        wave_order();       // the pushes of the last step come first
        if (lane < take) {
            const uint32_t ref = entry(n + lane);
            if (ref & kQLeaf) {
                uint32_t nt = 0;
                hit = leaf_anyhit<false>(sc, r, ref, nt);
            } else if (ref < n_groups) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint4 c = g[4 * (size_t)ref + k];
                    w[k] = qbox_hit(q, c) ? c.w : 0u;
                }
            }
        }
        if (__any(hit)) return true;
        wave_order();
        uint64_t live[4];
        int total = n;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            live[k] = __ballot(w[k] != 0u);
            total += (int)__popcll(live[k]);
        }
        flat = total > CAP;
        if (!flat) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (w[k] != 0u) entry(n + bits_below(live[k])) = w[k] & kRefMask;
                n += (int)__popcll(live[k]);
            }
        }
    }
    if (!flat) return false;
    uint32_t nb = 0, nt = 0;
    return qbvh_anyhit(sc, r, q, n_total, nb, nt);
}

__device__ __forceinline__ bool brute_anyhit(const Scene& sc, const Ray& r) {
    for (int64_t k = 0; k < sc.n_tris; ++k) {
        if (tri_anyhit(r, sc.tris, 48u * (uint32_t)k)) return true;
    }
    return false;
}

}  // namespace mcdi
