// Windowed Voigt line opacity, split by detuning: a far zone on the matrix
// cores and a near zone by direct evaluation.  pz_opacity.h holds the direct
// kernel, which plans with very dense lines take (see StarDev::split).
#pragma once

#include "pz_opacity.h"

namespace pz {

// ---------------------------------------------------------------- the split
// xfar[l] (dev_line_consts, dev_line_params) divides line l's window:
//   >= 0, finite: |x| >= xfar is the far zone (every depth has v >= PZ_FAR_V
//         and a <= PZ_FAR_AV v there), |x| < xfar the near zone;
//   +inf: the whole window is near (a non-finite parameter row, or the centre
//         test cuts the span of some depth inside the window);
//   -1:   the whole window is near and the line's damping ratio spans the
//         near and far wing tiers over depth (voigt_acc's SAFE form).
// Both passes evaluate x by the same float32 formula, so every (line, pixel)
// pair falls into exactly one zone.  Sums run in a fixed order: no atomics.

// Largest |x| of line l's near zone (a NaN xfar: the whole window).
__device__ __forceinline__ float near_reach(float xfar) { return xfar >= 0.0f ? xfar : INFINITY; }
__device__ __forceinline__ bool in_far_zone(float x, float xfar) { return xfar >= 0.0f && fabsf(x) >= xfar; }

// ------------------------------------------------------------------ far zone
// kappa[depth][pixel] = sum_(line, n) A_n[pixel][line] C_n[line][depth] with
// A_n = (xfar/x)^(2n) (0 outside the line's far zone) and far_poly's C_n: a
// matrix product whose inner index runs over lines and powers, on the float32
// matrix cores (16 x 16 x 4 tiles, float32 products and sums).
//
// A workgroup of FAR_WAVES wavefronts owns a tile of 32 pixels x all depths;
// wavefront w takes lines 4 (w + FAR_WAVES q) .. +3 of the tile's list, so
// each k-step of an MFMA is four lines: lane (r, c) = (lane / 16, lane % 16)
// forms A for pixel c and line r, and C for line r and depth c.  The operands
// live in registers from the parameter rows on: no LDS staging, no barrier
// until the wavefronts' partial sums are added (in order) at the end.
// Powers whose terms cannot reach 7e-8 of a line's opacity at the k-step's
// nearest pixel are left out (v >= 13: n <= 4; v >= 24: n <= 3; v >= 85:
// n <= 2), as are 16-pixel blocks with no far pixel.
typedef float f32x4 __attribute__((ext_vector_type(4)));
static constexpr int FAR_WAVES = 4;
static constexpr int FAR_NDT = (MAXD + 15) / 16;         // depth tiles
static constexpr int FAR_NPT = TILE / 16;                // pixel tiles
static constexpr float kFarU4 = 0.179f;                  // (5.5/13)^2
static constexpr float kFarU3 = 0.0525f;                 // (5.5/24)^2
static constexpr float kFarU2 = 0.0041f;                 // (5.5/86)^2

struct FarLds {
    f32x4 part[FAR_WAVES][FAR_NPT * FAR_NDT][WAVE];
};

// One k-step: u[t] the lane's (xfar/x)^2 for pixel tile t, row the parameter
// rows of the lane's line at depths 16 d + c.
template <int NT>
__device__ __forceinline__ void far_step(f32x4 (*acc)[FAR_NDT], const float* u, const bool* live, const float4* row,
                                         float xfar, int ndt) {
    float A[FAR_NPT][NT];
#pragma unroll
    for (int t = 0; t < FAR_NPT; ++t) {
        float p = u[t];
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            A[t][n] = p;
            p *= u[t];
        }
    }
#pragma unroll
    for (int d = 0; d < FAR_NDT; ++d)
        if (d < ndt) {
            const float sx = row[d].x * xfar;
            const float W = __builtin_amdgcn_rcpf(sx * sx);
            float C[NT];
            far_poly<NT>(PZ_FAR_H, row[d].y, W, row[d].w * W * kInvSqrtPiF, C);
#pragma unroll
            for (int t = 0; t < FAR_NPT; ++t)
                if (live[t]) {
#pragma unroll
                    for (int n = 0; n < NT; ++n)
                        acc[t][d] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[t][n], C[n], acc[t][d], 0, 0, 0);
                }
        }
}

__device__ __forceinline__ void dev_opacity_far(const StarDev& s, int tile, FarLds& lds) {
    const int lane = threadIdx.x % WAVE, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int c = lane % 16, r = lane / 16;
    const int p0 = tile * TILE;
    const int l0 = s.t32_first[tile], l1 = s.t32_last[tile];
    const int D = s.D, ndt = (D + 15) / 16;
    f32x4 acc[FAR_NPT][FAR_NDT];
#pragma unroll
    for (int t = 0; t < FAR_NPT; ++t)
#pragma unroll
        for (int d = 0; d < FAR_NDT; ++d) acc[t][d] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const char* rows = scalar_base(s.lp + (size_t)l0 * D);
    for (int b = l0 + 4 * wave; b < l1; b += 4 * FAR_WAVES) {
        const int l = min(b + r, l1 - 1);
        const float xf = b + r < l1 ? s.xfar[l] : -1.0f;
        const int lo = s.ln.ilo[l], hi = s.ln.ihi[l], ic = s.ln.ic[l];
        const float dl = s.ln.delta[l];
        float u[FAR_NPT];
        bool live[FAR_NPT];
        float um = 0.0f;
#pragma unroll
        for (int t = 0; t < FAR_NPT; ++t) {
            const int i = p0 + 16 * t + c;
            const float x = detuning(i - ic, dl, s.h_hi, s.h_lo);
            const float q = xf * __builtin_amdgcn_rcpf(x);
            u[t] = i >= lo && i <= hi && in_far_zone(x, xf) ? q * q : 0.0f;
            live[t] = wave_any(u[t] > 0.0f);
            um = fmaxf(um, u[t]);
        }
        if (!wave_any(um > 0.0f)) continue;
        // the rows of every lane (D x 16 B each; the plan keeps a tile's rows under 2^28 elements)
        float4 row[FAR_NDT];
        const unsigned e0 = (unsigned)((l - l0) * D);
#pragma unroll
        for (int d = 0; d < FAR_NDT; ++d)
            if (d < ndt) {
                row[d] = *(const float4*)(rows + (size_t)(e0 + (unsigned)min(16 * d + c, D - 1)) * 16u);
                if (!(xf >= 0.0f && xf < INFINITY)) row[d] = make_float4(1.0f, 0.0f, 0.0f, 0.0f);
            }
        const float x0 = xf >= 0.0f && xf < INFINITY ? xf : 1.0f;
        if (wave_any(um > kFarU4))
            far_step<PZ_FAR_N>(acc, u, live, row, x0, ndt);
        else if (wave_any(um > kFarU3))
            far_step<4>(acc, u, live, row, x0, ndt);
        else if (wave_any(um > kFarU2))
            far_step<3>(acc, u, live, row, x0, ndt);
        else
            far_step<2>(acc, u, live, row, x0, ndt);
    }
#pragma unroll
    for (int t = 0; t < FAR_NPT; ++t)
#pragma unroll
        for (int d = 0; d < FAR_NDT; ++d)
            if (d < ndt) lds.part[wave][t * FAR_NDT + d][lane] = acc[t][d];
    __syncthreads();
    for (int k = wave; k < FAR_NPT * FAR_NDT; k += FAR_WAVES) {
        const int t = k / FAR_NDT, d = k % FAR_NDT, j = 16 * d + c;
        if (d >= ndt) continue;
        f32x4 v = lds.part[0][k][lane];
#pragma unroll
        for (int w = 1; w < FAR_WAVES; ++w) v += lds.part[w][k][lane];
        // lane (r, c) holds pixels 4 r .. 4 r + 3 of the tile at depth c
        if (j < D) *(f32x4*)(s.kappa + (size_t)j * s.Npad + p0 + 16 * t + 4 * r) = v;
    }
}

// ----------------------------------------------------------------- near zone
// Wavefront w of a workgroup owns pixels 8 w .. 8 w + 7 of a tile and NG of its
// depth groups: lane (pixel p, depth q) = (lane % 8, lane / 8) holds depths
// 8 g + q, g < NG.  It scans the tile's lines 64 at a time (one per lane),
// keeps by ballot those whose near zone meets its pixels and takes them in
// order: x per pixel, then the NG depth groups in straight-line code, whose
// parameter rows come from L1/L2 (128 contiguous bytes a group).  Wavefronts
// are independent: no LDS staging and no barrier.  What bounds it is VALU
// issue; splitting the depths over NG-group wavefronts fills the chip on
// short grids and evens the last wave of long ones.
// With the centre test (CT) a lane adds a line only where z2 = v^2 + a^2 <=
// zmax of its (line, depth).
static constexpr int NEAR_G = 3;                          // depth groups per wavefront
__host__ __device__ constexpr int near_parts(int D) { return (D + 8 * NEAR_G - 1) / (8 * NEAR_G); }

template <int NP, bool CT, int NG>
__device__ __forceinline__ void wing_sums(float* acc, const float4* p, const float* z2, const float* zm,
                                          const float* T2, const float* W) {
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const float a = fmaf(p[g].w, wing_S<NP>(p[g].y, z2[g], T2, W), acc[g]);
        acc[g] = !CT || z2[g] <= zm[g] ? a : acc[g];
    }
}

template <int NG, bool CT>
__device__ __forceinline__ void near_line(float* acc, const float4* p, const float* zm, float x, bool safe,
                                          const float4* near_tab, const float4* pw) {
    float v[NG], z2[NG], amax = 0.0f, zmin = INFINITY, smax = 0.0f;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        v[g] = x * p[g].x;
        z2[g] = fmaf(v[g], v[g], p[g].y);
        amax = fmaxf(amax, p[g].y);
        smax = fmaxf(smax, fabsf(p[g].x));
        zmin = fminf(zmin, z2[g]);
    }
    if (!safe && wave_all(amax <= PZ_VOIGT_A2_SMALL && smax * fabsf(x) < PZ_NEAR_V)) {
        const bool full = wave_any(amax > PZ_VOIGT_A2_TINY);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const float a = full ? near_KH_acc<true>(acc[g], p[g].y, p[g].z, p[g].w, v[g], near_tab)
                                 : near_KH_acc<false>(acc[g], p[g].y, p[g].z, p[g].w, v[g], near_tab);
            acc[g] = !CT || z2[g] <= zm[g] ? a : acc[g];
        }
    } else if (!safe && wave_all(zmin >= PZ_VOIGT_WING_R2)) {
        // a line not flagged SAFE keeps each tier's pair products in range
        if (wave_all(zmin >= PZ_VOIGT_TIER3_R2))
            wing_sums<1, CT, NG>(acc, p, z2, zm, PZ_GH2_T2, PZ_GH2_W);
        else if (wave_all(zmin >= PZ_VOIGT_TIER2_R2))
            wing_sums<2, CT, NG>(acc, p, z2, zm, PZ_GH4_T2, PZ_GH4_W);
        else
            wing_sums<3, CT, NG>(acc, p, z2, zm, PZ_GH6_T2, PZ_GH6_W);
    } else {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const float z = CT ? zm[g] : 0.0f;
            acc[g] = safe ? voigt_acc<CT, true>(acc[g], p[g].y, p[g].z, p[g].w, v[g], pw, z)
                          : voigt_acc<CT, false>(acc[g], p[g].y, p[g].z, p[g].w, v[g], pw, z);
        }
    }
}

// Adds the near zone to the far zone's kappa (written before).
template <int NG, bool CT>
__device__ __forceinline__ void dev_opacity_near(const StarDev& s, int tile, int part, const float4* near_tab,
                                                 const float4* pw) {
    const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
    const int D = s.D;
    const int p0 = __builtin_amdgcn_readfirstlane(tile * TILE + 8 * wave);
    const int i = p0 + lane % 8, j0 = part * (8 * NG) + lane / 8;
    const int l0 = s.t32_first[tile], l1 = s.t32_last[tile];
    const float inv_h = 1.0f / s.h_hi;
    unsigned off[NG];                                     // byte offset of a lane's depths in a row
    float acc[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        off[g] = (unsigned)min(j0 + 8 * g, D - 1) * 16u;
        acc[g] = 0.0f;
    }
    for (int b = l0; b < l1; b += WAVE) {
        const int l = min(b + lane, l1 - 1);
        const float xf = s.xfar[l];
        int lo = s.ln.ilo[l], hi = s.ln.ihi[l];
        const int ic = s.ln.ic[l];
        const float dl = s.ln.delta[l];
        float reach = near_reach(xf);
        if (CT) reach = fminf(reach, s.xlim[l] * (1.0f + 1e-5f));
        // pixels with |x| < reach lie within (reach + reach^2) / h + 1/2 of the anchor
        const float w = fmaf(reach, reach, reach) * inv_h + 2.0f;
        if (reach < 0.5f && w < 1.0e6f) {
            lo = max(lo, ic - (int)w);
            hi = min(hi, ic + (int)w);
        }
        unsigned long long m = __builtin_amdgcn_ballot_w64(b + lane < l1 && lo <= p0 + 7 && hi >= p0);
        while (m) {
            const int k = __builtin_ctzll(m);
            m &= m - 1;
            const float x = detuning(i - __builtin_amdgcn_readlane(ic, k), __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dl), k)),
                                     s.h_hi, s.h_lo);
            const float rc = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(reach), k));
            const bool safe = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(xf), k)) < 0.0f;
            if (i >= __builtin_amdgcn_readlane(lo, k) && i <= __builtin_amdgcn_readlane(hi, k) && fabsf(x) < rc) {
                const size_t e = (size_t)(b + k) * D;
                const char* row = (const char*)(s.lp + e);
                float4 p[NG];
                float zm[NG];
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    p[g] = *(const float4*)(row + off[g]);
                    zm[g] = CT ? *(const float*)((const char*)(s.zmax + e) + off[g] / 4u) : 0.0f;
                }
                near_line<NG, CT>(acc, p, zm, x, safe, near_tab, pw);
            }
        }
    }
    if (i < s.N) {
#pragma unroll
        for (int g = 0; g < NG; ++g)
            if (j0 + 8 * g < D) s.kappa[(size_t)(j0 + 8 * g) * s.Npad + i] += acc[g];
    }
}

}  // namespace pz
