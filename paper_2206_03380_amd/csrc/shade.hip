// Per-pixel Monte Carlo direct illumination on gfx950: forward (c_d, c_s and
// shadow-ray hit bits) and the adjoint of the detached estimator.
//
// One lane owns one pixel and loops over its samples; each sample draws one
// light-technique direction and one BSDF-technique direction (cosine or GGX
// visible normals, chosen with probability q), weights both with the balance
// heuristic over the three techniques and traces one shadow ray per
// direction above the horizon (paper: section 3.1, section 4.1, appendix D).
// The marginal CDF of the probe is staged in LDS; the per-pixel frame, view
// vector and visible-normal frame are set up in FP64 once per pixel (FP64
// FMA runs at the FP32 rate on CDNA, and it removes the ill-conditioning of
// the tangent frame when the view is close to the normal).
#include <hip/hip_runtime.h>
#include <math.h>

// Multiply-adds are fused only within one source expression, never across
// statements, so a sample's arithmetic rounds the same way in every loop that
// evaluates it (the staged forward's walk over live samples, the decision
// dump's full walk, the serving kernel's lockstep walk) and their results
// agree bit for bit.  (Set before the shared headers, whose inline functions
// are compiled here; the triangle test turns contraction off itself.)
#pragma clang fp contract(on)

#include "device_common.h"
#include "shade_common.h"

namespace mcdi {

namespace {

// visible-normal sample (Heitz 2018), local frame
// (r, sp, cp: sqrt(u1), sin and cos of 2 pi u2)
__device__ __forceinline__ float3 sample_vndf(const Pixel& P, float r, float sp, float cp) {
    const float a1 = r * cp;
    float a2 = r * sp;
    const float s = 0.5f * (1.0f + P.vh.z);
    a2 = (1.0f - s) * sqrtf(fmaxf(0.0f, 1.0f - a1 * a1)) + s * a2;
    const float az = sqrtf(fmaxf(0.0f, 1.0f - a1 * a1 - a2 * a2));
    const float3 nh = f3(a1 * P.t1x + a2 * P.t2v.x + az * P.vh.x, a1 * P.t1y + a2 * P.t2v.y + az * P.vh.y,
                         a2 * P.t2v.z + az * P.vh.z);
    const float3 ne = normalize(f3(P.alpha * nh.x, P.alpha * nh.y, fmaxf(0.0f, nh.z)));
    const float vn = dot(P.Vl, ne);
    return (2.0f * vn) * ne - P.Vl;
}

struct Sample {
    float3 wl;     // local direction
    float3 w;      // world direction
    float pL;      // light-technique density
    int texel;     // probe texel index i*W + j
    float x, y;    // continuous texel coordinates (phi W / 2 pi, theta H / pi)
    float4 tx;     // the texel's (r, g, b, pdf), read once per sample
};

struct FwdAcc {
    float3 cd, cs;
};

struct BwdAcc {
    float3 gkd;
    float gm, gr;
    float3 gnl;  // d/dn in the local frame
};

// Light technique: piecewise-constant 2D distribution over the probe.
// Returns false when the sample has no density (direction at a pole).
// How each stage draws a light sample:
//  kDrawGen  ray generation: whether the density is positive, from the
//            texels' 2-bit density classes (the density table for tiny
//            densities): the sample's density itself is not used there;
//  kDrawFwd  forward shading: the texel's radiance and density, kept for the
//            evaluation;
//  kDrawBwd  adjoint: the density from the radiance table (the evaluation
//            reads that line again) and always the binary row search, which
//            needs fewer registers than the adjoint has to spare.
// The other two read the row's candidates in one go (cdf_find_row).
enum DrawMode { kDrawGen, kDrawFwd, kDrawBwd };

template <int MODE>
__device__ __forceinline__ bool draw_light(const ShadeArgs& A, const Pixel& P, const float* s_marg, uint4 r0,
                                           Sample& S) {
    const int H = A.env.H, W = A.env.W;
    const float x0 = u01(r0.x), x1 = u01(r0.y);
    const int i = cdf_find_padded(s_marg, search_size(H), x0);
    const float* crow = A.env.cond + (size_t)i * (W + 1);
    float c0, c1;
    int j;
    if (MODE != kDrawBwd) {
        j = cdf_find_row(crow, A.env.guide + (size_t)i * (A.env.G + 1), A.env.G, x1, c0, c1);
    } else {
        j = cdf_find_guided(crow, A.env.guide + (size_t)i * (A.env.G + 1), A.env.G, x1);
        c0 = crow[j];
        c1 = crow[j + 1];
    }
    const float m0 = s_marg[i], m1 = s_marg[i + 1];
    S.y = (float)i + (x0 - m0) / (m1 - m0);
    S.x = (float)j + (x1 - c0) / (c1 - c0);
    const float v = div_small(S.y, (float)H, 1.0f / (float)H);
    const float u = div_small(S.x, (float)W, 1.0f / (float)W);
    float st, ct, sp, cp;
    sincospif(v, &st, &ct);
    sincospif(2.0f * u, &sp, &cp);
    S.w = f3(st * cp, ct, st * sp);
    S.texel = i * W + j;
    bool tiny = false;
    if (MODE == kDrawFwd) {
        S.tx = A.env.tex[S.texel];
    } else if (MODE == kDrawGen) {
        // generation only asks whether the density is positive: the
        // texel's class answers it except for tiny densities (class 2)
        const uint32_t cls = (A.env.dclass[S.texel >> 2] >> (2 * (S.texel & 3))) & 3u;
        tiny = cls == 2u;
        S.tx.w = tiny ? A.env.pdf[S.texel] : (float)cls;
    } else {
        S.tx.w = A.env.tex[S.texel].w;
    }
    // (generation: a normal density over at most 2 pi^2 is positive)
    if (MODE == kDrawGen && !tiny) S.pL = st > 0.0f ? S.tx.w : 0.0f;
    else S.pL = st > 0.0f ? S.tx.w / (2.0f * kPi * kPi * st) : 0.0f;
    S.wl = f3(dot(S.w, P.t), dot(S.w, P.b), dot(S.w, P.n));
    return S.pL > 0.0f;
}

// BSDF technique: cosine lobe with probability q, else GGX visible normals.
__device__ __forceinline__ bool draw_bsdf(const Pixel& P, uint4 r0, uint4 r1, Sample& S) {
    const float x2 = u01(r0.z), x4 = u01(r1.x), x5 = u01(r1.y);
    const bool cosl = x2 < P.q;
    // both lobes map the unit disk: a wave usually draws from both
    const float rr = sqrtf(x4);
    float sp, cp;
    sincospif(2.0f * x5, &sp, &cp);
    if (cosl) {
        S.wl = f3(rr * cp, rr * sp, sqrtf(fmaxf(0.0f, 1.0f - x4)));
    } else {
        S.wl = sample_vndf(P, rr, sp, cp);
    }
    S.w = normalize(S.wl.x * P.t + S.wl.y * P.b + S.wl.z * P.n);
    S.pL = 0.0f;
    S.texel = -1;
    return cosl;
}

// probe texel (nearest) of a BSDF-sampled direction and its light density
template <bool KEEP>
__device__ __forceinline__ void bsdf_texel(const ShadeArgs& A, bool light_on, Sample& S) {
    const int H = A.env.H, W = A.env.W;
    const float rho = sqrtf(S.w.x * S.w.x + S.w.z * S.w.z);
    const float th = atan2f(rho, S.w.y);
    float ph = atan2f(S.w.z, S.w.x);
    if (ph < 0.0f) ph += 2.0f * kPi;
    S.y = th * ((float)H * kInvPi);
    S.x = ph * ((float)W * (0.5f * kInvPi));
    const int ti = min((int)S.y, H - 1);
    const int tj = min((int)S.x, W - 1);
    S.texel = ti * W + tj;
    if (KEEP) {
        S.tx = A.env.tex[S.texel];
        if (light_on && rho > 0.0f) S.pL = S.tx.w / (2.0f * kPi * kPi * rho);
    } else if (light_on && rho > 0.0f) {
        S.pL = A.env.tex[S.texel].w / (2.0f * kPi * kPi * rho);
    }
}

// where the adjoint puts probe-gradient records of non-hot texels: the tile's
// record region and its LDS fill counter (base NULL: direct global atomics)
struct RecSink {
    float4* base;
    uint32_t* count;
};

// one record (n float4s) appended to the tile's region: one LDS counter
// atomic per wave; the region holds every record the tile can make
template <int NQ>
__device__ __forceinline__ void append_record(const RecSink& rs, const float4 (&q)[NQ]) {
    const uint64_t act = __ballot(1);
    const int lane = (int)__lane_id();
    const int leader = __ffsll((unsigned long long)act) - 1;
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(rs.count, (uint32_t)__popcll(act));
    base = (uint32_t)__shfl((int)base, leader);
    const uint32_t at = base + (uint32_t)__popcll(act & ((1ull << lane) - 1ull));
#pragma unroll
    for (int k = 0; k < NQ; ++k) rs.base[(size_t)NQ * at + k] = q[k];
}

// probe-gradient contribution (v0, v1, v2) of one texel: hot texels go to
// the workgroup's LDS copy, the rest to the tile's records (or straight to
// global memory when there are none)
// maybe_hot false: the texel's density rules it out of the hot set (its slot
// is not read)
__device__ __forceinline__ void scatter_texel(const ShadeArgs& A, int texel, float v0, float v1, float v2,
                                              float* s_hot, const RecSink& rs, bool maybe_hot = true) {
    const int slot = maybe_hot ? A.env.hot_slot[texel] : -1;
    if (slot >= 0) {
        atomicAdd(s_hot + 3 * slot + 0, v0);
        atomicAdd(s_hot + 3 * slot + 1, v1);
        atomicAdd(s_hot + 3 * slot + 2, v2);
    } else if (v0 == 0.0f && v1 == 0.0f && v2 == 0.0f) {
        // nothing to add (a shadowed sample with tau = 1, a zero tap weight)
    } else if (rs.base) {
        const float4 q[1] = {make_float4(__uint_as_float((uint32_t)texel), v0, v1, v2)};
        append_record<1>(rs, q);
    } else {
        float* ge = A.g_env + 3 * (size_t)texel;
        atomicAdd(ge + 0, v0);
        atomicAdd(ge + 1, v1);
        atomicAdd(ge + 2, v2);
    }
}

// balance-heuristic denominator of a sample: the densities of the techniques
// in use at its direction
__device__ __forceinline__ float mis_density(const Pixel& P, const Sample& S) {
    const float3 hl = normalize(P.Vl + S.wl);
    const float D = ggx_D(hl.z, hl.x * hl.x + hl.y * hl.y, P.a2);
    const float pcos = S.wl.z * kInvPi;
    const float pggx = P.nov_pos ? P.G1V * D / (4.0f * P.nov) : 0.0f;
    return S.pL + P.bsdf_w * (P.q * pcos + (1.0f - P.q) * pggx);
}

// FROZEN: the sample was drawn from another pixel state, whose density
// (Pt_frozen) weighs it; P and S.wl evaluate it
template <bool BWD, bool BIL, bool FROZEN = false>
__device__ __forceinline__ void eval_sample(const ShadeArgs& A, const Pixel& P, const Sample& S, float Hv,
                                            float invspp, FwdAcc& fa, BwdAcc& ba, float3 Ud, float3 Us,
                                            float* s_hot, const RecSink& rs, float Pt_frozen = 0.0f) {
    const float NoL = S.wl.z;
    const float3 hl = normalize(P.Vl + S.wl);
    const float NoH = hl.z;
    const float s2 = hl.x * hl.x + hl.y * hl.y;
    const float VoH = dot(P.Vl, hl);
    const float D = ggx_D(NoH, s2, P.a2);
    const float pcos = NoL * kInvPi;
    const float pggx = P.nov_pos ? P.G1V * D / (4.0f * P.nov) : 0.0f;
    // balance heuristic over the techniques in use
    const float Pt = FROZEN ? Pt_frozen : S.pL + P.bsdf_w * (P.q * pcos + (1.0f - P.q) * pggx);
    const float w = Hv / Pt;
    float3 L;
    float pdf_uv = 0.0f;   // nearest lookup: the texel's density (pdf table)
    if (BIL) {
        const Taps T = bilinear_taps(A.env, S.x, S.y);
        L = T.w[0] * texel_rgb(A.env, T.t[0]) + T.w[1] * texel_rgb(A.env, T.t[1]) +
            T.w[2] * texel_rgb(A.env, T.t[2]) + T.w[3] * texel_rgb(A.env, T.t[3]);
    } else {
        // the forward keeps the texel from the draw; the adjoint, short of
        // registers, reads it again
        const float4 tx = BWD ? A.env.tex[S.texel] : S.tx;
        L = f3(tx.x, tx.y, tx.z);
        pdf_uv = tx.w;
    }
    const float kdiff = (1.0f - P.m) * kInvPi * NoL;
    float S_ = 0.0f, Fw = 0.0f, G2 = 0.0f, lamL = 0.0f, t2L = 0.0f;
    float3 F = f3(0, 0, 0);
    if (P.nov_pos) {
        t2L = smith_t2(NoL);
        lamL = smith_lambda(t2L, P.a2);
        G2 = 1.0f / (1.0f + P.lamV + lamL);
        S_ = D * G2 / (4.0f * P.nov);
        const float omv = 1.0f - VoH;
        const float o2 = omv * omv;
        Fw = o2 * o2 * omv;
        F = f3(P.F0.x + (1.0f - P.F0.x) * Fw, P.F0.y + (1.0f - P.F0.y) * Fw, P.F0.z + (1.0f - P.F0.z) * Fw);
    }
    if (!BWD) {
        fa.cd = fa.cd + (kdiff * w) * L;
        fa.cs = fa.cs + (S_ * w) * f3(F.x * L.x, F.y * L.y, F.z * L.z);
        return;
    }
    const float K = w * invspp;
    // probe texel gradient: the coefficient of L_c, times the tap weight
    const float cdc = kdiff * K, csc = S_ * K;
    if (A.g_env) {
        const float v0 = Ud.x * cdc + Us.x * F.x * csc;
        const float v1 = Ud.y * cdc + Us.y * F.y * csc;
        const float v2 = Ud.z * cdc + Us.z * F.z * csc;
        if (BIL) {
            // taps recomputed from the coordinates: cheaper than keeping
            // them live across the BSDF terms
            const Taps T = bilinear_taps(A.env, S.x, S.y);
            if (rs.base) {
                // one record per sample (base, fractions, coefficient), split
                // into the four taps by the env-scatter pass; no LDS hot
                // sums here: twelve contended LDS float atomics per sample
                // cost more than the record
                if (v0 != 0.0f || v1 != 0.0f || v2 != 0.0f) {
                    const float4 q[2] = {make_float4(__uint_as_float((uint32_t)T.base), T.fx, T.fy, 0.0f),
                                         make_float4(v0, v1, v2, 0.0f)};
                    append_record<2>(rs, q);
                }
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    scatter_texel(A, T.t[k], T.w[k] * v0, T.w[k] * v1, T.w[k] * v2, s_hot, rs);
            }
        } else {
            // hot texels have pdf > W H / kHotMax (the hot-set rule); half that
            // bound keeps the test free of rounding questions
            const bool maybe_hot = pdf_uv > 0.5f * ((float)A.env.W * (float)A.env.H / (float)kHotMax);
            scatter_texel(A, S.texel, v0, v1, v2, s_hot, rs, maybe_hot);
        }
    }
    const float udL = Ud.x * L.x + Ud.y * L.y + Ud.z * L.z;
    const float usL = Us.x * L.x + Us.y * L.y + Us.z * L.z;
    const float uskdL = Us.x * P.kd.x * L.x + Us.y * P.kd.y * L.y + Us.z * P.kd.z * L.z;
    const float usFL = Us.x * F.x * L.x + Us.y * F.y * L.y + Us.z * F.z * L.z;
    const float omF = 1.0f - Fw;
    ba.gkd = ba.gkd + (P.m * omF * S_ * K) * f3(Us.x * L.x, Us.y * L.y, Us.z * L.z);
    ba.gm += -NoL * kInvPi * K * udL + omF * S_ * K * (uskdL - 0.04f * usL);
    // diffuse part of d/dn: (1-m)/pi * udL * K * w_l
    float3 gn = ((1.0f - P.m) * kInvPi * udL * K) * S.wl;
    if (P.nov_pos) {
        const float a = P.alpha, a2 = P.a2;
        const float B = a2 * NoH * NoH + s2;
        const float dDda = D * (2.0f / a - 4.0f * a * NoH * NoH / B);
        const float t2V = smith_t2(P.nov);
        const float sqV = sqrtf(1.0f + a2 * t2V), sqL = sqrtf(1.0f + a2 * t2L);
        const float dlamV_da = a * t2V / (2.0f * sqV), dlamL_da = a * t2L / (2.0f * sqL);
        const float G2s = G2 * G2;
        const float dSda = (dDda * G2 - D * G2s * (dlamV_da + dlamL_da)) / (4.0f * P.nov);
        const float dSdr = P.r_active ? dSda * 2.0f * P.r : 0.0f;
        ba.gr += usFL * K * dSdr;
        const float dlamV_dx = -a2 / (2.0f * P.nov * P.nov * P.nov * sqV);
        const float dlamL_dx = -a2 / (2.0f * NoL * NoL * NoL * sqL);
        const float dSdV = -D * G2s * dlamV_dx / (4.0f * P.nov) - S_ / P.nov;
        const float dSdL = -D * G2s * dlamL_dx / (4.0f * P.nov);
        const float dSdH = D * 4.0f * (1.0f - a2) * NoH / B * G2 / (4.0f * P.nov);
        const float c = usFL * K;
        gn = gn + (c * dSdV) * P.Vl + (c * dSdL) * S.wl + (c * dSdH) * hl;
    }
    ba.gnl = ba.gnl + gn;
}

// bit k of the result = bit 2k of x (k < 16)
__device__ __forceinline__ uint32_t even_bits(uint32_t x) {
    x &= 0x55555555u;
    x = (x | (x >> 1)) & 0x33333333u;
    x = (x | (x >> 2)) & 0x0F0F0F0Fu;
    x = (x | (x >> 4)) & 0x00FF00FFu;
    x = (x | (x >> 8)) & 0x0000FFFFu;
    return x;
}

// the marginal CDF in LDS: H + 1 entries, padded for the search (and to 16 bytes)
__host__ __device__ inline int marg_entries(int H) {
    const int p = search_size(H);
    return ((p > H + 1 ? p : H + 1) + 3) & ~3;
}
__device__ __forceinline__ void stage_marg(const ShadeArgs& A, float* s_marg) {
    const int H = A.env.H, n = marg_entries(H);
    for (int k = threadIdx.x; k < n; k += blockDim.x) s_marg[k] = k <= H ? A.env.marg[k] : 1.0f;
}

// ---------------------------------------------------------------------------
// The three stages work on one tile of kBlock pixels per workgroup.  The
// staged kernels run tile = blockIdx.x; the serving kernel pulls tiles of
// many requests from a queue and runs the stages back to back.
// ---------------------------------------------------------------------------

// 1) ray generation: the directions of every sample above the horizon,
//    compacted into the tile's ray region (LDS counter, no global atomics);
//    hit words of the tile's pixels are cleared; returns the ray count
//    (valid in thread 0 after the final barrier, in *s_cnt for all).
template <bool COUNT>
__device__ __forceinline__ void gen_tile(const ShadeArgs& A, int64_t tile, float4* region, uint32_t* hitbits,
                                         const float* s_marg, int* s_cnt) {
    const int64_t N = A.g.n;
    const int64_t pix = tile * kBlock + threadIdx.x;
    const bool active = pix < N;
    const int spp = A.spp;
    const int words = (2 * spp + 31) >> 5;
    const bool light_on = (*A.env.light_enabled != 0) && !(A.flags & MCDI_FLAG_LIGHT_OFF);
    const bool trace = A.tau != 0.0f && region != nullptr;
    bool nonfinite = false;
    Pixel P;
    P.valid = false;
    if (active) {
        for (int k = 0; k < words; ++k) hitbits[k * N + pix] = 0u;
        P = setup_pixel(A, pix, nonfinite);
        if (P.valid) A.origins[pix] = make_float4(P.o.x, P.o.y, P.o.z, 0.0f);
    }
    const bool go = P.valid && trace;
    const int64_t hw = (int64_t)A.g.height * A.g.width;
    const uint32_t view = active ? (uint32_t)(pix / hw) : 0u;
    const uint32_t piv = active ? (uint32_t)(pix - (int64_t)view * hw) : 0u;
    const uint32_t vid = (uint32_t)A.g.view_base + view;
    const uint32_t k0 = (uint32_t)A.seed, k1 = (uint32_t)(A.seed >> 32);
    const int lane = __lane_id();
    uint32_t c_rays = 0, c_culled = 0;
    uint32_t lw = 0u;   // live bits of the current word
    for (int s = 0; s < spp; ++s) {
        uint4 r0 = make_uint4(0, 0, 0, 0), r1 = r0;
        if (go) {
            r0 = philox10(make_uint4(piv, vid, (uint32_t)s, 0u), k0, k1);
            r1 = philox10(make_uint4(piv, vid, (uint32_t)s, 1u), k0, k1);
        }
        for (int tech = 0; tech < 2; ++tech) {
            bool want = false;
            Sample S;
            if (go) {
                bool has = true;
                if (tech == 0) has = light_on && draw_light<kDrawGen>(A, P, s_marg, r0, S);
                else if (P.bsdf_w != 0.0f) draw_bsdf(P, r0, r1, S);
                else has = false;
                want = has && S.wl.z > 0.0f;
                if (has && !want) ++c_culled;
            }
            const uint64_t bal = __ballot(want);
            if (bal == 0ull) continue;
            int base = 0;
            if (lane == 0) base = atomicAdd(s_cnt, (int)__popcll(bal));
            base = __shfl(base, 0);
            if (want) {
                const int slot = 2 * s + tech;
                const uint32_t tag = (uint32_t)threadIdx.x | ((uint32_t)slot << 8);
                region[base + bits_below(bal)] = make_float4(S.w.x, S.w.y, S.w.z, __uint_as_float(tag));
                lw |= 1u << (slot & 31);
                ++c_rays;
            }
        }
        if (A.live && active && ((s & 15) == 15 || s == spp - 1)) {
            A.live[(s >> 4) * N + pix] = lw;
            lw = 0u;
        }
    }
    if (COUNT) {
        const uint32_t a = wave_sum(c_rays), b = wave_sum(c_culled);
        const uint32_t v = wave_sum(P.valid ? 1u : 0u), nf = wave_sum(nonfinite ? 1u : 0u);
        if (lane == 0) {
            atomicAdd(&A.stats->rays_traced, (unsigned long long)a);
            atomicAdd(&A.stats->samples_culled, (unsigned long long)b);
            atomicAdd(&A.stats->valid_pixels, (unsigned long long)v);
            atomicAdd(&A.stats->invalid_pixels, (unsigned long long)nf);
        }
    }
}

// 2) any-hit traversal of the tile's ray region over the 4-wide hierarchy.
//    Lanes that finish a ray take the next one from the region (one LDS atomic
//    per wave per refill); box steps and triangle steps run in separate phases
//    so a wave keeps its lanes on the same code (while-while traversal with
//    dynamic fetch).
//
//    Per lane: the next node (a wide node to visit; a leaf reference that
//    waits for the pending slot; kWideNone, the walk is over or the lane holds
//    no ray) and one postponed leaf (its reference, 0 = none).  Testing one
//    triangle of a leaf with more advances its reference by 3: the first
//    index grows by one and the rest drops by one.
//
//    What bounds it: instruction issue (93% of the vector issue slots at four
//    cycles an instruction, in a room of 1.0M triangles and on a 101k-triangle
//    surface) and, where the nodes come from the L1 cache, its
//    gathers: 64 lanes at 64 addresses take it about 45 cycles whether a lane
//    fetches 4 bytes or 16 and whether the four loads of a node share a line
//    (measured), so a wide node costs 180 of them beside 110 cycles of its
//    CU's vector issue.  The root's first kTopNodes descendants are therefore
//    read from LDS (L1 accesses per box test, the triangles' included, 1.16 ->
//    0.59 in the room, 1.13 -> 0.96 on the surface), the
//    visit order comes with the records instead of by a fifth load, and the
//    loop holds one walk: a ray whose stack overflows, and it alone, walks the
//    binary nodes after the visits of the step.
//    Shadow rays, before (two walks in the loop, a separate order word, two
//    pending leaves, no hoisted nodes) -> after: 4.2M pixels at 32 spp in the
//    room 10.6 -> 7.1 ms (5.4 with the big triangles' SAH subtree), 1.05M pixels at
//    12 spp on a 102k-triangle surface 2.36 -> 1.70 ms, 201k pixels at 16 spp
//    on a 45k-triangle one 545 -> 385 us, 4096 pixels at 4 spp 45 -> 30 us.
//
// Pending references of the wide traversal, per lane, in LDS: row k of the
// workgroup's lane t at [k * kBlock + t] (lanes of a wave hit distinct banks
// whatever their stack depths).  Row 0 holds kWideNone, so that popping an
// empty stack ends the walk without a test.  Up to kStack + 1 references
// after a visit's pushes (the visit pops one again), and three spare rows for
// its last stores.  Eight workgroups per CU fit, with the hoisted nodes.
constexpr int kStack = 13, kStackRows = 1 + kStack + 4;
// references a full stack hands to private memory at a time, and how many it
// holds (a ray that needs more walks the binary nodes from the root)
constexpr uint32_t kSpill = 8, kSpillMax = 32;
// stands for them at the bottom of the stack: a leaf reference past every
// triangle array that no record holds
constexpr uint32_t kMoreRef = leaf_ref((1u << 26) - 1u, 2u);
static_assert(kMoreRef != kEmptyRef && kMoreRef != kWideNone && (kMoreRef & kRefMask) == kMoreRef, "");

// a struct of words as lane l holds it
template <typename T>
__device__ __forceinline__ T read_lane(const T& v, int l) {
    struct Words { uint32_t w[sizeof(T) / 4]; };
    Words u = __builtin_bit_cast(Words, v);
#pragma unroll
    for (uint32_t k = 0; k < sizeof(T) / 4; ++k) u.w[k] = (uint32_t)__builtin_amdgcn_readlane((int)u.w[k], l);
    return __builtin_bit_cast(T, u);
}

// Where a walk's rays come from and its hits go to: take() gives ray idx and
// its tag, which hit() gets back.
struct TileFeed {      // a tile's generated shadow rays, and the hit bits
    const float4* R;
    const float4* origins;   // of the tile's first pixel
    uint32_t* hitbits;       // the same
    int64_t N;
    __device__ __forceinline__ uint32_t take(int idx, float3& o, float3& d) const {
        const float4 rr = R[idx];
        const uint32_t tag = __float_as_uint(rr.w);   // pixel within the tile | sample slot << 8
        const float4 oo = origins[tag & 255u];
        o = f3(oo.x, oo.y, oo.z);
        d = f3(rr.x, rr.y, rr.z);
        return tag;
    }
    __device__ __forceinline__ void hit(uint32_t tag) const {
        const uint32_t slot = tag >> 8;
        atomicOr(hitbits + (int64_t)(slot >> 5) * N + (tag & 255u), 1u << (slot & 31));
    }
};
__device__ __forceinline__ TileFeed tile_feed(const ShadeArgs& A, int64_t tile, const float4* R, uint32_t* hitbits) {
    return TileFeed{R, A.origins + tile * kBlock, hitbits + tile * kBlock, A.g.n};
}
struct QueryFeed {     // planes [3][n] from a workgroup's first ray, and its bytes
    const float *o, *d;
    int64_t n;
    uint8_t* bytes;
    __device__ __forceinline__ uint32_t take(int idx, float3& ro, float3& rd) const {
        ro = f3(o[idx], o[n + idx], o[2 * n + idx]);
        rd = f3(d[idx], d[n + idx], d[2 * n + idx]);
        bytes[idx] = 0;      // the lane that takes the ray is the one that reports it
        return (uint32_t)idx;
    }
    __device__ __forceinline__ void hit(uint32_t tag) const { bytes[tag] = 1; }
};

// TAIL: the longest rays bound the launch, so a full stack goes to private
// memory and a wave's last kTailRays rays, kTailRounds rounds after the last was
// taken, are walked by the whole wave (query_kernel says what that gives).
constexpr int kTailRays = 4, kTailRounds = 6;
template <bool COUNT, bool TAIL, typename Feed>
__device__ __forceinline__ void trace_tile(const Scene& sc, const Feed& feed, int count, int* s_next,
                                           uint32_t* s_stack, uint4* s_top, mcdi_stats* stats) {
    const int n_total = sc.nodes[0].escape;
    const uint32_t n_tris = (uint32_t)sc.n_tris;
    const QFrame F = *sc.frame;
    // a hierarchy that failed the builder's check (never for a valid tree):
    // every ray walks the binary nodes
    const bool flat = sc.info->wide_bad != 0;
    // nodes as a buffer resource: 32-bit offsets, and a load past the end
    // returns zeros instead of reading out of bounds
    const __amdgpu_buffer_rsrc_t grs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)sc.groups, (short)0, (int)sc.group_bytes, kBufferWord3);
    for (int k = threadIdx.x; k < 4 * kTopNodes; k += kBlock) s_top[k] = reinterpret_cast<const uint4*>(sc.top)[k];
    s_stack[threadIdx.x] = kWideNone;
    __syncthreads();
    // the stack's first free row as a byte offset
    constexpr uint32_t kRow = 4u * kBlock, kOverflow = (1u + kStack + 1u) * kRow;
    const uint32_t sp0 = 4u * threadIdx.x + kRow, sp_end = 4u * threadIdx.x + kOverflow;
    uint32_t sp = sp0;
    auto row = [&](uint32_t at) -> uint32_t& {
        return *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(s_stack) + at);
    };
    const int lane = __lane_id();
    bool exhausted = n_total <= 0;   // uniform: no ray is left to take
    Ray ray;
    QRay qray;
    uint32_t oct = 0u;     // the ray's octant
    // (every wide walk ends: the builder checked that each internal child
    // reference is larger than its parent's index and smaller than the node
    // count)
    uint32_t node = kWideNone, p0 = 0u;
    uint32_t tag = 0u;
    bool restart = false;  // the stack overflowed
    int rounds = 0;        // since the last ray was taken
    uint32_t c_hits = 0, c_box = 0, c_tri = 0, c_bstep = 0, c_tstep = 0;   // steps: lane 0 only
    uint32_t c_blane = 0;
    auto report = [&]() {
        feed.hit(tag);
        if (COUNT) ++c_hits;
    };
    // The lane's stack is full: its kSpill oldest references go to the lane's
    // private memory, and kMoreRef takes their place in row 1 (row 0 stays).
    uint32_t priv[1 + kSpillMax];   // how many (valid below a kMoreRef in row 1), and the references
    auto unload = [&]() {
        const bool again = row(sp0) == kMoreRef;
        const uint32_t had = again ? priv[0] : 0u;
        if (had + kSpill > kSpillMax) {
            restart = true;
            return;
        }
        uint32_t from = sp0 + (again ? kRow : 0u), to = sp0 + kRow;
        for (uint32_t k = 1; k <= kSpill; ++k, from += kRow) priv[had + k] = row(from);
        priv[0] = had + kSpill;
        // (at least kStack + 1 - kSpill references move down, in increasing
        // rows, not above where they were)
        for (; from < sp; from += kRow, to += kRow) row(to) = row(from);
        row(sp0) = kMoreRef;
        sp = to;
    };
    // the walk came down to kMoreRef (the stack is empty): the newest of them back
    auto reload = [&]() {
        const uint32_t left = priv[0] - kSpill;
        priv[0] = left;
        sp = sp0;
        if (left != 0u) {
            row(sp) = kMoreRef;
            sp += kRow;
        }
        for (uint32_t k = 1; k <= kSpill; ++k, sp += kRow) row(sp) = priv[left + k];
        sp -= kRow;
        node = row(sp) & kRefMask;
        p0 = 0u;
    };
    // scheduling knobs: refill batch, node visits per phase check, and the
    // phase hand-over ratios (the box phase ends once four times the lanes
    // stuck on leaves are as many as the walkers, the triangle phase once the
    // lanes free to walk are more than twice the testers).  Measured on the
    // room below: 3, 4, 5, 6 and 7 visits 6.3, 5.3, 5.4, 5.8 and 6.3 ms; the
    // other knobs a step up or down stay within 3%.
    constexpr int kRefillMin = 16, kBoxSteps = 4, kBoxSwitch4 = 1, kTriSwitch2 = 4;
    while (true) {
        // refill when a quarter of the wave is idle, or when nobody is busy
        if (!exhausted) {
            const bool idle = node == kWideNone && p0 == 0u;
            const uint64_t need = __ballot(idle);
            const int n_need = (int)__popcll(need);
            if (n_need >= kRefillMin) {
                int b = 0;
                if (lane == 0) b = atomicAdd(s_next, n_need);
                b = __builtin_amdgcn_readfirstlane(b);
                exhausted = b + n_need >= count;
                const int idx = b + bits_below(need);
                if (idle && idx < count) {
                    float3 o, d;
                    tag = feed.take(idx, o, d);
                    ray = make_ray(o, d);
                    qray = make_qray(ray, F);
                    oct = ray_octant(d);
                    node = flat ? kWideNone : kRefTop;   // the root, hoisted node 0
                    restart = flat;
                    sp = sp0;
                }
            }
        }
        // box phase: lanes visit wide nodes; a lane whose next node is a leaf
        // waits for its pending slot
        while (true) {
#pragma unroll
            for (int step = 0; step < kBoxSteps; ++step) {
                const bool walking = (int)node >= 0;
                if (COUNT && __any(walking) && lane == 0) ++c_bstep;
                if (COUNT && walking) ++c_blane;
                if (walking) {
                    // one wide node: four child records from one 64-byte
                    // segment, in LDS when the node is hoisted
                    uint4 c[4];
                    if (node & kRefTop) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) c[k] = s_top[4u * (node & (kRefTop - 1u)) + k];
                    } else {
                        const uint32_t off = node * 64u;
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            c[k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(grs, off + 16u * k, 0, 0));
                    }
                    // a missed child's reference becomes 0 (no kRefLive
                    // bit: the push below does not keep it)
                    uint32_t w[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if (COUNT && (c[k].w & kRefMask) != kEmptyRef) ++c_box;
                        w[k] = qbox_hit(qray, c[k]) ? c[k].w : 0u;
                    }
                    // farther child of each split after the nearer one
                    // (the pushed-last is popped first): within each pair,
                    // then the pairs
                    const bool s0 = split_swaps(oct, c[1].w), s1 = split_swaps(oct, c[2].w),
                               sT = split_swaps(oct, c[0].w);
                    const uint32_t a0 = s0 ? w[1] : w[0], a1 = s0 ? w[0] : w[1];
                    const uint32_t a2 = s1 ? w[3] : w[2], a3 = s1 ? w[2] : w[3];
                    const uint32_t ws[4] = {sT ? a2 : a0, sT ? a3 : a1, sT ? a0 : a2, sT ? a1 : a3};
                    // every hit child is pushed: each record is stored at
                    // the first free row and the row is kept if the child
                    // was hit; then the top is popped as the next node
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        row(sp) = ws[k];
                        sp += ((ws[k] >> 30) & 1u) * kRow;
                    }
                    if (sp > sp_end) {
                        if (TAIL) unload();
                        else restart = true;
                    }
                    sp -= kRow;
                    node = row(sp) & kRefMask;
                    // a leaf on top goes to the pending slot if that is free,
                    // and the next entry is popped
                    if (p0 == 0u && (int)node < 0 && node != kWideNone) {
                        p0 = node;
                        sp -= kRow;
                        node = row(sp) & kRefMask;
                    }
                    if (restart) node = kWideNone;
                }
            }
            if (__any(restart)) {
                // the stack was full: these rays walk the binary tree from
                // the root instead (the same answer, more steps)
                if (restart) {
                    uint32_t nb = 0, nt = 0;
                    if (qbvh_anyhit<COUNT>(sc, ray, qray, n_total, nb, nt)) report();
                    c_box += nb;
                    c_tri += nt;
                    restart = false;
                    node = kWideNone;
                    p0 = 0u;
                }
            }
            const uint64_t walk = __ballot((int)node >= 0);
            if (walk == 0ull) break;
            const uint64_t stuck = __ballot(p0 != 0u && (int)node < 0);
            if (4 * __popcll(stuck) >= kBoxSwitch4 * __popcll(walk)) break;
        }
        // triangle phase: one triangle of the pending leaf per lane and step;
        // it ends when no leaf is pending, or when lanes that could walk but
        // hold no leaf outnumber the lanes testing
        while (true) {
            const bool test = p0 != 0u;
            if (!__any(test)) break;
            if (COUNT && lane == 0) ++c_tstep;
            if (test) {
                const uint32_t t = (p0 >> 2) & 0x03FFFFFFu;
                bool h = false;
                if (t < n_tris) {
                    if (COUNT) ++c_tri;
                    h = tri_anyhit(ray, sc.tris, t * 48u);
                } else if (TAIL && p0 == kMoreRef) {   // (another reference past the triangle array tests nothing)
                    reload();
                }
                if (h) {
                    report();
                    node = kWideNone;
                    p0 = 0u;
                } else if ((p0 & 3u) != 0u) {
                    p0 += 3u;
                } else {
                    p0 = 0u;
                    if ((int)node < 0 && node != kWideNone) {   // the leaf that waited
                        p0 = node;
                        sp -= kRow;
                        node = row(sp) & kRefMask;
                    }
                }
            }
            const uint64_t testing = __ballot(p0 != 0u);
            const uint64_t free_ = __ballot(p0 == 0u && (int)node >= 0);
            if (2 * __popcll(free_) > kTriSwitch2 * __popcll(testing)) break;
        }
        if (exhausted) {
            uint64_t left = __ballot(node != kWideNone || p0 != 0u);
            if (left == 0ull) break;
            // the last rays of the wave, each by all its lanes from the root
            // (the lanes' stacks are dropped)
            if (TAIL && ++rounds > kTailRounds && (int)__popcll(left) <= kTailRays) {
                for (; left != 0ull; left &= left - 1ull) {
                    const int l = (int)__ffsll((unsigned long long)left) - 1;
                    const bool h = wave_anyhit<kBlock, kStackRows * 64>(sc, read_lane(ray, l), read_lane(qray, l), n_total,
                                                                        s_stack + (threadIdx.x & ~63u));
                    if (h && lane == l) report();
                }
                break;
            }
        }
    }
    if (COUNT) {
        const uint32_t h = wave_sum(c_hits), bx = wave_sum(c_box), tr = wave_sum(c_tri), bl = wave_sum(c_blane);
        if (lane == 0) {
            atomicAdd(&stats->box_lanes, (unsigned long long)bl);
            atomicAdd(&stats->rays_hit, (unsigned long long)h);
            atomicAdd(&stats->box_tests, (unsigned long long)bx);
            atomicAdd(&stats->tri_tests, (unsigned long long)tr);
            atomicAdd(&stats->box_slots, 64ull * c_bstep);
            atomicAdd(&stats->tri_slots, 64ull * c_tstep);
        }
    }
}

// 3) evaluation: forward values or the adjoint, from the hit bits.  For the
//    adjoint, s_hot must be zeroed before and flushed after (hot_flush).
//    BIL: bilinear probe lookup (MCDI_FLAG_BILINEAR) instead of the nearest
//    texel.
// words per sample of the decision dump: 3, or 9 with the sampled world
// directions (MCDI_FLAG_DUMP_DIRS)
constexpr uint32_t kNanBits = 0x7FC00000u;
__device__ __forceinline__ int dump_stride(const ShadeArgs& A) { return (A.flags & MCDI_FLAG_DUMP_DIRS) ? 9 : 3; }

// FROZEN (forward only): samples, densities, lobe choice and visibility from
// the G-buffer A.g, the samples evaluated with the planes A.e_*.
// LOCKSTEP: the lanes step through every sample pair together, skipping a pair
// blocked twice over in place (the persistent serving kernel, whose launches
// ran a quarter slower with the per-lane walk below).
template <bool BWD, bool DUMP, bool BIL, bool FROZEN = false, bool LOCKSTEP = false>
__device__ __forceinline__ void shade_tile(const ShadeArgs& A, int64_t tile, const float* s_marg, float* s_hot,
                                           const RecSink& rs) {
    const int64_t N = A.g.n;
    const int64_t pix = tile * kBlock + threadIdx.x;
    const int spp = A.spp;
    const bool light_on = (*A.env.light_enabled != 0) && !(A.flags & MCDI_FLAG_LIGHT_OFF);
    const bool trace = A.tau != 0.0f;
    if (pix >= N) return;
    bool nonfinite;
    const Pixel P = setup_pixel(A, pix, nonfinite);
    Pixel Pe;
    if (FROZEN) {
        ShadeArgs Ae = A;
        Ae.g.nrm = A.e_nrm;
        Ae.g.kd = A.e_kd;
        Ae.g.korm = A.e_korm;
        bool nf;
        Pe = setup_pixel(Ae, pix, nf);
    }
    if (!P.valid || (FROZEN && !Pe.valid)) {
        if (!BWD) {
            for (int c = 0; c < 3; ++c) { A.c_d[c * N + pix] = 0.0f; A.c_s[c * N + pix] = 0.0f; }
        } else {
            for (int c = 0; c < 3; ++c) {
                A.g_kd[c * N + pix] = 0.0f; A.g_korm[c * N + pix] = 0.0f; A.g_nrm[c * N + pix] = 0.0f;
            }
        }
        if (DUMP) {
            const int st = dump_stride(A);
            uint32_t* d = A.decisions + (size_t)pix * spp * st;
            for (int s = 0; s < spp; ++s) {
                d[st * s] = kNone; d[st * s + 1] = kNone; d[st * s + 2] = 0u;
                for (int k = 3; k < st; ++k) d[st * s + k] = kNanBits;
            }
        }
        return;
    }
    const int64_t hw = (int64_t)A.g.height * A.g.width;
    const uint32_t view = (uint32_t)(pix / hw), piv = (uint32_t)(pix - (int64_t)view * hw);
    const uint32_t vid = (uint32_t)A.g.view_base + view;
    const uint32_t k0 = (uint32_t)A.seed, k1 = (uint32_t)(A.seed >> 32);
    const float invspp = 1.0f / (float)spp;
    float3 Ud = f3(0, 0, 0), Us = f3(0, 0, 0);
    if (BWD) {
        Ud = f3(A.g_cd[pix], A.g_cd[N + pix], A.g_cd[2 * N + pix]);
        Us = f3(A.g_cs[pix], A.g_cs[N + pix], A.g_cs[2 * N + pix]);
    }
    FwdAcc fa{f3(0, 0, 0), f3(0, 0, 0)};
    BwdAcc ba{f3(0, 0, 0), 0.0f, 0.0f, f3(0, 0, 0)};
    // With tau = 1 a blocked sample is weighted by H = 0 and adds nothing
    // (the incident radiance is the probe's times H, appendix A): its hit
    // bit (set only for a traced, blocked ray) skips it before it is drawn.
    // A lane walks only its pixel's sample pairs that are not blocked twice
    // over (in increasing order, so the sums are those of the full loop), so
    // a wavefront runs as many pair steps as its busiest lane rather than
    // spp.  The decision dump draws every sample and skips only the
    // evaluation.
    const bool skip_blocked = !DUMP && A.tau == 1.0f;
    if (!DUMP && !FROZEN && !LOCKSTEP && A.live) {
        // the live bits name the samples the estimator evaluates: a lane
        // draws and evaluates only those (and with tau = 1 only those not
        // blocked), pair by pair in the same increasing (sample, technique)
        // order; the two samples of a pair share the first Philox block
        for (int s0 = 0; s0 < spp; s0 += 16) {
            const uint32_t bits = A.hitbits_in[(s0 >> 4) * N + pix];
            uint32_t need = A.live[(s0 >> 4) * N + pix];
            if (skip_blocked) need &= ~bits;
            uint32_t todo = even_bits(need | (need >> 1));
            while (todo) {
                const int k = __ffs(todo) - 1;
                todo &= todo - 1u;
                const int s = s0 + k;
                const uint32_t pair = need >> (2 * k), hit = bits >> (2 * k);
                const uint4 r0 = philox10(make_uint4(piv, vid, (uint32_t)s, 0u), k0, k1);
                if (pair & 1u) {
                    Sample S;
                    draw_light<BWD ? kDrawBwd : kDrawFwd>(A, P, s_marg, r0, S);
                    const float Hv = (hit & 1u) ? 1.0f - A.tau : 1.0f;
                    eval_sample<BWD, BIL>(A, P, S, Hv, invspp, fa, ba, Ud, Us, s_hot, rs);
                }
                if (pair & 2u) {
                    Sample S;
                    const uint4 r1 = philox10(make_uint4(piv, vid, (uint32_t)s, 1u), k0, k1);
                    draw_bsdf(P, r0, r1, S);
                    bsdf_texel<!BWD>(A, light_on, S);
                    const float Hv = (hit & 2u) ? 1.0f - A.tau : 1.0f;
                    eval_sample<BWD, BIL>(A, P, S, Hv, invspp, fa, ba, Ud, Us, s_hot, rs);
                }
            }
        }
    } else {
        for (int s0 = 0; s0 < spp; s0 += 16) {
            const uint32_t bits = A.hitbits_in[(s0 >> 4) * N + pix];   // pairs s0 .. s0 + 15
            uint32_t todo = (spp - s0 >= 16) ? 0xFFFFu : (1u << (spp - s0)) - 1u;
            if (skip_blocked && !LOCKSTEP) todo &= ~even_bits(bits & (bits >> 1));
            while (todo) {
                const int s = s0 + __ffs(todo) - 1;
                todo &= todo - 1u;
                if (LOCKSTEP && skip_blocked && ((bits >> ((2 * s) & 31)) & 3u) == 3u) continue;
                const uint4 r0 = philox10(make_uint4(piv, vid, (uint32_t)s, 0u), k0, k1);
                const uint4 r1 = philox10(make_uint4(piv, vid, (uint32_t)s, 1u), k0, k1);
                uint32_t rec0 = kNone, rec1 = kNone;
                uint32_t rec2 = kDecValid | (P.nov_pos ? kDecNovPos : 0u);
                float3 dir[2] = {f3(__uint_as_float(kNanBits), 0.0f, 0.0f), f3(__uint_as_float(kNanBits), 0.0f, 0.0f)};
                for (int tech = 0; tech < 2; ++tech) {
                    if (skip_blocked && ((bits >> ((2 * s + tech) & 31)) & 1u)) continue;
                    Sample S;
                    if (tech == 0) {
                        if (!light_on) continue;
                        const bool has = draw_light<BWD ? kDrawBwd : kDrawFwd>(A, P, s_marg, r0, S);
                        rec0 = (uint32_t)S.texel;
                        if (DUMP) dir[0] = S.w;
                        if (!has) { rec2 |= kDecLCull; continue; }
                    } else {
                        if (P.bsdf_w == 0.0f) continue;
                        if (draw_bsdf(P, r0, r1, S)) rec2 |= kDecLobeCos;
                        if (DUMP) dir[1] = S.w;
                    }
                    if (!(S.wl.z > 0.0f)) { rec2 |= tech ? kDecBCull : kDecLCull; continue; }
                    if (tech == 1) {
                        bsdf_texel<!BWD>(A, light_on, S);
                        rec1 = (uint32_t)S.texel;
                    }
                    float Hv = 1.0f;
                    if (trace) {
                        const int bitpos = 2 * s + tech;
                        rec2 |= tech ? kDecBTraced : kDecLTraced;
                        if ((bits >> (bitpos & 31)) & 1u) {
                            Hv = 1.0f - A.tau;
                            rec2 |= tech ? kDecBHit : kDecLHit;
                        }
                    }
                    // H = 0: no incident radiance, whatever the probe holds there
                    if (Hv == 0.0f) continue;
                    if (FROZEN) {
                        // the sample's direction in the evaluation frame (the
                        // sampled local direction itself where the frame is the same)
                        Sample Se = S;
                        if (!(Pe.n.x == P.n.x && Pe.n.y == P.n.y && Pe.n.z == P.n.z))
                            Se.wl = f3(dot(S.w, Pe.t), dot(S.w, Pe.b), dot(S.w, Pe.n));
                        eval_sample<BWD, BIL, true>(A, Pe, Se, Hv, invspp, fa, ba, Ud, Us, s_hot, rs, mis_density(P, S));
                    } else {
                        eval_sample<BWD, BIL>(A, P, S, Hv, invspp, fa, ba, Ud, Us, s_hot, rs);
                    }
                }
                if (DUMP) {
                    const int st = dump_stride(A);
                    uint32_t* d = A.decisions + ((size_t)pix * spp + s) * st;
                    d[0] = rec0; d[1] = rec1; d[2] = rec2;
                    if (st == 9) {
                        for (int t = 0; t < 2; ++t) {
                            d[3 + 3 * t] = __float_as_uint(dir[t].x);
                            d[4 + 3 * t] = __float_as_uint(dir[t].y);
                            d[5 + 3 * t] = __float_as_uint(dir[t].z);
                        }
                    }
                }
            }
        }
    }
    if (!BWD) {
        for (int c = 0; c < 3; ++c) {
            A.c_d[c * N + pix] = comp(fa.cd, c) * invspp;
            A.c_s[c * N + pix] = comp(fa.cs, c) * invspp;
        }
    } else {
        A.g_kd[pix] = ba.gkd.x; A.g_kd[N + pix] = ba.gkd.y; A.g_kd[2 * N + pix] = ba.gkd.z;
        A.g_korm[pix] = 0.0f; A.g_korm[N + pix] = ba.gr; A.g_korm[2 * N + pix] = ba.gm;
        const float il = 1.0f / P.nlen;
        const float3 gw = (ba.gnl.x * il) * P.t + (ba.gnl.y * il) * P.b;
        A.g_nrm[pix] = gw.x; A.g_nrm[N + pix] = gw.y; A.g_nrm[2 * N + pix] = gw.z;
    }
}

__device__ __forceinline__ void hot_zero(float* s_hot) {
    for (int k = threadIdx.x; k < 3 * kHotMax; k += blockDim.x) s_hot[k] = 0.0f;
}

// one global atomic per touched hot slot (call after a barrier)
__device__ __forceinline__ void hot_flush(const ShadeArgs& A, const float* s_hot) {
    if (!A.g_env) return;
    const int n_hot = min(*A.env.n_hot, kHotMax);
    for (int k = threadIdx.x; k < 3 * n_hot; k += blockDim.x) {
        const float v = s_hot[k];
        if (v != 0.0f) atomicAdd(A.g_env + 3 * (size_t)A.env.hot_texel[k / 3] + (k % 3), v);
    }
}

__device__ __forceinline__ float4* tile_region(const ShadeArgs& A, int64_t tile) {
    return A.rays ? A.rays + (size_t)tile * (size_t)(2 * A.spp * kBlock) : nullptr;
}

template <bool COUNT>
__global__ __launch_bounds__(kBlock) void gen_rays_kernel(ShadeArgs A, uint32_t* hitbits) {
    extern __shared__ float s_marg[];
    __shared__ int s_cnt;
    stage_marg(A, s_marg);
    if (threadIdx.x == 0) s_cnt = 0;
    __syncthreads();
    gen_tile<COUNT>(A, blockIdx.x, tile_region(A, blockIdx.x), hitbits, s_marg, &s_cnt);
    __syncthreads();
    if (threadIdx.x == 0) A.ray_count[blockIdx.x] = s_cnt;
}

// Traversal order of the tiles: a counting sort by ray count, most rays
// first, so that the longest workgroups start first and the short ones fill
// the end of the launch (longest-processing-time-first).  One workgroup;
// counts are bucketed by 8 rays (beyond 8184 rays a tile is just "long").
// The order of tiles within a bucket is arbitrary: traversal results do not
// depend on it.
constexpr int kOrderBuckets = 1024;

__global__ __launch_bounds__(1024) void order_tiles_kernel(const int32_t* __restrict__ cnt, int64_t n,
                                                           int32_t* __restrict__ order) {
    __shared__ int h[kOrderBuckets];
    const int tid = threadIdx.x;
    h[tid] = 0;
    __syncthreads();
    auto bucket = [](int c) { return kOrderBuckets - 1 - min(max(c, 0) >> 3, kOrderBuckets - 1); };
    for (int64_t t = tid; t < n; t += 1024) atomicAdd(&h[bucket(cnt[t])], 1);
    __syncthreads();
    // exclusive scan over the buckets (bucket 0 = the most rays)
    int v = h[tid];
    for (int off = 1; off < kOrderBuckets; off <<= 1) {
        const int a = tid >= off ? h[tid - off] : 0;
        __syncthreads();
        h[tid] += a;
        __syncthreads();
    }
    h[tid] -= v;
    __syncthreads();
    for (int64_t t = tid; t < n; t += 1024) {
        const int pos = atomicAdd(&h[bucket(cnt[t])], 1);
        order[pos] = (int32_t)t;
    }
}

// eight waves per SIMD (the hardware's limit): 64 registers per lane, 20 KB
// of LDS per workgroup.
// Workgroup b traces part b % parts of the b / parts-th tile's rays.
template <bool COUNT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8))) void trace_rays_kernel(
    ShadeArgs A, uint32_t* hitbits, int parts) {
    __shared__ int s_next;
    __shared__ uint32_t s_stack[kStackRows * kBlock];
    __shared__ uint4 s_top[4 * kTopNodes];
    const int rank = (int)blockIdx.x / parts, part = (int)blockIdx.x - rank * parts;
    const int tile = __builtin_amdgcn_readfirstlane(A.tile_order ? A.tile_order[rank] : rank);
    if (tile < 0 || tile >= (int)gridDim.x / parts) return;   // uniform: the whole workgroup reads the same entry
    const int all = __builtin_amdgcn_readfirstlane(A.ray_count[tile]);
    const int chunk = ((all + parts - 1) / parts + 63) & ~63, first = part * chunk;
    if (first >= all) return;
    if (threadIdx.x == 0) s_next = 0;
    __syncthreads();
    trace_tile<COUNT, false>(A.scene, tile_feed(A, tile, tile_region(A, tile) + first, hitbits), min(chunk, all - first),
                      &s_next, s_stack, s_top, A.stats);
}

// Any-hit queries over the 4-wide hierarchy: workgroup b walks rays
// [b chunk, (b + 1) chunk) as it would a tile's, a lane one or a few rays, so
// the longest rays bound it: at 400k incoherent rays against 296k triangles the
// one-lane walk of the binary nodes took 268 us, this walk 290 (one ray whose
// stack overflowed walked the binary nodes for 100 us alone), with the full
// stack handed to private memory 190, and with a wave's last rays walked by all
// its lanes 145; 127 at six waves per SIMD, which spill nothing (eight: 140,
// five: 135).  20k rays 191 -> 73, 1M 428 -> 204, 4M 1233 -> 500; 400k against
// 590 triangles 61 -> 52, against a room of 1.0M 358 -> 189.  The last four
// rays six rounds after the last was taken: two rays or four rounds more are
// within 10%, no wait costs short walks (590 triangles: 86 us).  The shading
// kernels' walk, bound by throughput, does without either: the registers that
// they take cost it 25%.
constexpr int kQueryChunk = 4096;   // rays of a workgroup, at most (1024: 4M rays 600 us, 4096: 530)
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6))) void query_kernel(
    Scene sc, const float* o, const float* d, int64_t n, uint8_t* hit, int chunk) {
    __shared__ int s_next;
    __shared__ uint32_t s_stack[kStackRows * kBlock];
    __shared__ uint4 s_top[4 * kTopNodes];
    const int64_t first = (int64_t)blockIdx.x * chunk;
    const int count = (int)min((int64_t)chunk, n - first);
    if (sc.nodes[0].escape <= 0) {      // an empty scene
        for (int k = threadIdx.x; k < count; k += kBlock) hit[first + k] = 0;
        return;
    }
    if (threadIdx.x == 0) s_next = 0;
    __syncthreads();
    trace_tile<false, true>(sc, QueryFeed{o + first, d + first, n, hit + first}, count, &s_next, s_stack, s_top, nullptr);
}

template <bool BWD, bool DUMP, bool BIL>
__device__ __forceinline__ void shade_body(const ShadeArgs& A) {
    extern __shared__ float smem[];
    __shared__ uint32_t s_rec;
    float* s_marg = smem;
    float* s_hot = smem + marg_entries(A.env.H);
    stage_marg(A, s_marg);
    if (BWD) hot_zero(s_hot);
    if (threadIdx.x == 0) s_rec = 0u;
    __syncthreads();
    const RecSink rs{(BWD && A.rec) ? A.rec + (size_t)blockIdx.x * A.rec_region * (BIL ? 2 : 1) : nullptr, &s_rec};
    shade_tile<BWD, DUMP, BIL>(A, blockIdx.x, s_marg, s_hot, rs);
    if (BWD) {
        __syncthreads();
        hot_flush(A, s_hot);
        if (A.rec && threadIdx.x == 0) A.rec_count[blockIdx.x] = s_rec;
    }
}

// Four waves per SIMD (at most 128 VGPRs) for every variant except the
// bilinear adjoint, which spills at that bound and runs faster at three.
template <bool BWD, bool DUMP, bool BIL>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void shade_kernel(ShadeArgs A) {
    shade_body<BWD, DUMP, BIL>(A);
}

// forward with frozen sampling (a test instantiation: finite differences of
// the estimator with its samples held fixed)
template <bool BIL>
__global__ __launch_bounds__(kBlock) void shade_frozen_kernel(ShadeArgs A) {
    extern __shared__ float smem[];
    stage_marg(A, smem);
    __syncthreads();
    shade_tile<false, false, BIL, true>(A, blockIdx.x, smem, nullptr, RecSink{nullptr, nullptr});
}

__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3))) void shade_bwd_bilinear_kernel(ShadeArgs A) {
    shade_body<true, false, true>(A);
}

// ---------------------------------------------------------------------------
// Serving: one persistent launch over the tiles of many requests.  Every
// workgroup takes the next tile from a global counter and runs generation,
// traversal, the forward evaluation and (for gradient requests) the adjoint
// on it; it stops when the tiles run out, so every wave exits.  Four waves
// per SIMD (128 VGPRs, 112 bytes spilled): left to itself the compiler takes
// 171 registers for the adjoint's stretch and the whole launch runs at two
// waves, the traversal's included; on the serving mix four waves served 16%
// more requests per second, five and six (more spills) fewer.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void serve_kernel(const ServeItem* items, int n_items, int64_t total_tiles,
                                                       int* tile_counter, float4* scratch, int spp_max) {
    extern __shared__ float smem[];
    __shared__ int s_tile, s_item, s_cnt, s_next;
    __shared__ uint32_t s_stack[kStackRows * kBlock];
    __shared__ uint4 s_top[4 * kTopNodes];
    float* s_hot = smem;                     // 3 * kHotMax
    float* s_marg = smem + 3 * kHotMax;      // marg_entries(H) of the current item
    float4* region = scratch + (size_t)blockIdx.x * (size_t)(2 * spp_max * kBlock);
    while (true) {
        if (threadIdx.x == 0) {
            const int t = atomicAdd(tile_counter, 1);
            int lo = 0, hi = n_items;           // item with first_global <= t
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (items[mid].first_global <= t) lo = mid; else hi = mid;
            }
            s_tile = t;
            s_item = lo;
            s_cnt = 0;
            s_next = 0;
        }
        __syncthreads();
        const int64_t t = s_tile;
        if (t >= total_tiles) break;
        const ServeItem& it = items[s_item];
        const ShadeArgs& A = it.args;
        const int64_t tile = it.first_tile + (t - it.first_global);
        stage_marg(A, s_marg);
        __syncthreads();
        float4* reg = A.tau != 0.0f ? region : nullptr;
        gen_tile<false>(A, tile, reg, it.hitbits, s_marg, &s_cnt);
        __syncthreads();
        if (reg)
            trace_tile<false, false>(A.scene, tile_feed(A, tile, reg, it.hitbits), s_cnt, &s_next, s_stack, s_top, nullptr);
        __syncthreads();
        const bool bil = (A.flags & MCDI_FLAG_BILINEAR) != 0;
        if (bil) shade_tile<false, false, true, false, true>(A, tile, s_marg, s_hot, RecSink{nullptr, nullptr});
        else shade_tile<false, false, false, false, true>(A, tile, s_marg, s_hot, RecSink{nullptr, nullptr});
        if (A.g_cd) {
            hot_zero(s_hot);
            __syncthreads();
            if (bil) shade_tile<true, false, true, false, true>(A, tile, s_marg, s_hot, RecSink{nullptr, nullptr});
            else shade_tile<true, false, false, false, true>(A, tile, s_marg, s_hot, RecSink{nullptr, nullptr});
            __syncthreads();
            hot_flush(A, s_hot);
        }
        __syncthreads();
    }
}

__global__ void serve_reset(int* tile_counter) { *tile_counter = 0; }

__global__ void trace_kernel(Scene sc, const float* o, const float* d, int64_t n, uint8_t* hit, bool brute) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const Ray r = make_ray(f3(o[k], o[n + k], o[2 * n + k]), f3(d[k], d[n + k], d[2 * n + k]));
    uint32_t nb = 0, nt = 0;
    const bool h = brute ? brute_anyhit(sc, r)
                         : qbvh_anyhit(sc, r, make_qray(r, *sc.frame), sc.nodes[0].escape, nb, nt);
    hit[k] = h ? 1 : 0;
}

}  // namespace

static unsigned n_blocks(const ShadeArgs& a) { return (unsigned)((a.g.n + kBlock - 1) / kBlock); }

// Workgroups that share one tile's rays in the traversal.  256 CUs hold 2048
// of its workgroups; a launch with fewer tiles leaves CUs idle while each
// lane walks up to 2 spp rays one after another, so its tiles are split until
// they fill the chip once, at most down to one ray per lane.  Measured when
// the rule was made (traversal, one part against this rule): 16 tiles at 4 spp
// 137 -> 45 us, 382 tiles at 8 spp 398 -> 150 us, 1572 tiles at 16 spp 883 ->
// 545 us; filling the chip twice or four times over gives 189 and 235 us at
// 382 tiles, and splitting launches that fill it already costs (8192 tiles at
// 12 spp: 2.36 ms whole, 2.51 in halves; 16384 tiles at 32 spp: 10.6 whole,
// 11.1 in halves).
static int trace_parts(const ShadeArgs& a) {
    constexpr unsigned kSlots = 2048;
    const unsigned tiles = n_blocks(a), most = 2u * (unsigned)a.spp;
    const unsigned p = (kSlots + tiles - 1) / tiles;
    return (int)(p < most ? p : most);
}

static size_t marg_lds(const ShadeArgs& a) { return sizeof(float) * (size_t)marg_entries(a.env.H); }

hipError_t launch_gen_rays(const ShadeArgs& a, uint32_t* hitbits, hipStream_t s) {
    if (a.stats)
        hipLaunchKernelGGL((gen_rays_kernel<true>), dim3(n_blocks(a)), dim3(kBlock), marg_lds(a), s, a, hitbits);
    else
        hipLaunchKernelGGL((gen_rays_kernel<false>), dim3(n_blocks(a)), dim3(kBlock), marg_lds(a), s, a, hitbits);
    return hipGetLastError();
}

hipError_t launch_order_tiles(const int32_t* ray_count, int64_t n_tiles, int32_t* order, hipStream_t s) {
    hipLaunchKernelGGL(order_tiles_kernel, dim3(1), dim3(1024), 0, s, ray_count, n_tiles, order);
    return hipGetLastError();
}

hipError_t launch_trace_rays(const ShadeArgs& a, uint32_t* hitbits, hipStream_t s) {
    const int parts = trace_parts(a);
    const dim3 g(n_blocks(a) * (unsigned)parts);
    if (a.stats) hipLaunchKernelGGL((trace_rays_kernel<true>), g, dim3(kBlock), 0, s, a, hitbits, parts);
    else hipLaunchKernelGGL((trace_rays_kernel<false>), g, dim3(kBlock), 0, s, a, hitbits, parts);
    return hipGetLastError();
}

hipError_t launch_shade_fwd(const ShadeArgs& a, hipStream_t s) {
    const bool dump = (a.flags & MCDI_FLAG_DUMP) != 0, bil = (a.flags & MCDI_FLAG_BILINEAR) != 0;
    const dim3 g(n_blocks(a)), b(kBlock);
    if (dump && bil) hipLaunchKernelGGL((shade_kernel<false, true, true>), g, b, marg_lds(a), s, a);
    else if (dump) hipLaunchKernelGGL((shade_kernel<false, true, false>), g, b, marg_lds(a), s, a);
    else if (bil) hipLaunchKernelGGL((shade_kernel<false, false, true>), g, b, marg_lds(a), s, a);
    else hipLaunchKernelGGL((shade_kernel<false, false, false>), g, b, marg_lds(a), s, a);
    return hipGetLastError();
}

hipError_t launch_serve(const ServeItem* items_dev, int n_items, int64_t total_tiles, int* tile_counter,
                        float4* scratch, int spp_max, int n_workgroups, int max_H, hipStream_t s) {
    hipLaunchKernelGGL(serve_reset, dim3(1), dim3(1), 0, s, tile_counter);
    const size_t lds = sizeof(float) * (3 * kHotMax + (size_t)marg_entries(max_H));
    hipLaunchKernelGGL(serve_kernel, dim3(n_workgroups), dim3(kBlock), lds, s, items_dev, n_items, total_tiles,
                       tile_counter, scratch, spp_max);
    return hipGetLastError();
}

hipError_t launch_shade_fwd_frozen(const ShadeArgs& a, hipStream_t s) {
    const dim3 g(n_blocks(a)), b(kBlock);
    if (a.flags & MCDI_FLAG_BILINEAR) hipLaunchKernelGGL(shade_frozen_kernel<true>, g, b, marg_lds(a), s, a);
    else hipLaunchKernelGGL(shade_frozen_kernel<false>, g, b, marg_lds(a), s, a);
    return hipGetLastError();
}

hipError_t launch_shade_bwd(const ShadeArgs& a, hipStream_t s) {
    const size_t lds = marg_lds(a) + sizeof(float) * 3 * kHotMax;
    if (a.flags & MCDI_FLAG_BILINEAR)
        hipLaunchKernelGGL(shade_bwd_bilinear_kernel, dim3(n_blocks(a)), dim3(kBlock), lds, s, a);
    else
        hipLaunchKernelGGL((shade_kernel<true, false, false>), dim3(n_blocks(a)), dim3(kBlock), lds, s, a);
    return hipGetLastError();
}

// mode 0: the binary nodes, 1: every triangle, 2: the 4-wide nodes
hipError_t launch_trace(const Scene& sc, const float* o, const float* d, int64_t n, uint8_t* hit, int mode,
                        hipStream_t s) {
    if (n == 0) return hipSuccess;
    if (mode == 2) {
        const int64_t slots = 2048, fill = ((n + slots - 1) / slots + 63) & ~(int64_t)63;
        const int chunk = (int)(fill < kBlock ? kBlock : fill > kQueryChunk ? kQueryChunk : fill);
        hipLaunchKernelGGL(query_kernel, dim3((unsigned)((n + chunk - 1) / chunk)), dim3(kBlock), 0, s, sc, o, d, n, hit,
                           chunk);
        return hipGetLastError();
    }
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(trace_kernel, dim3((unsigned)blocks), dim3(256), 0, s, sc, o, d, n, hit, mode == 1);
    return hipGetLastError();
}

}  // namespace mcdi
