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
// A workgroup owns 16 NPT pixels x all depths; of its nw wavefronts, w takes
// lines 4 (w + nw q) .. +3 of the tile's list, so each k-step of an MFMA is
// four lines: lane (r, c) = (lane / 16, lane % 16) forms A for pixel c and
// line r, and C for line r and depth c.  The operands live in registers from
// the parameter rows on, the next step's loads in flight: no LDS staging, no
// barrier until the wavefronts' partial sums are added (in a fixed order).
// Powers whose terms cannot reach 7e-8 of a line's opacity at the k-step's
// nearest pixel are left out (v >= 13: n <= 4; v >= 24: n <= 3; v >= 85:
// n <= 2), as are 16-pixel blocks with no far pixel.
typedef float f32x4 __attribute__((ext_vector_type(4)));
static constexpr int FAR_NDT = (MAXD + 15) / 16;         // depth tiles
static constexpr float kFarU4 = 0.179f;                  // (5.5/13)^2
static constexpr float kFarU3 = 0.0525f;                 // (5.5/24)^2
static constexpr float kFarU2 = 0.0041f;                 // (5.5/86)^2
// Whether a grid of n 32-pixel tiles takes 64 pixels per workgroup.
__host__ __device__ constexpr bool far_wide(int n) { return n >= 4096; }

// Pixels per workgroup: NPT 16-pixel blocks share a line's coefficients and
// loads.  Four (64 pixels) where the grid fills the chip, two below that.
template <int NPT>
constexpr int far_waves() {
    return NPT == 2 ? 8 : 4;
}
template <int NPT>
struct FarLds {
    f32x4 part[far_waves<NPT>() / 2][FAR_NDT][WAVE];
};

// The window fields and parameter rows of one k-step (four lines).
struct FarStep {
    float xf, dl;
    int lo, hi, ic;
    float4 row[FAR_NDT];
};

__device__ __forceinline__ void far_load(const StarDev& s, const char* rows, int l0, int l1, int b, int r, int c, int ndt,
                                         FarStep& q) {
    const int l = min(b + r, l1 - 1);
    q.xf = s.xfar[l];
    q.lo = s.ln.ilo[l];
    q.hi = s.ln.ihi[l];
    q.ic = s.ln.ic[l];
    q.dl = s.ln.delta[l];
    if (b + r >= l1) q.xf = -1.0f;
    // the plan keeps a tile's rows under 2^28 elements
    const unsigned e0 = (unsigned)((l - l0) * s.D);
#pragma unroll
    for (int d = 0; d < FAR_NDT; ++d)
        if (d < ndt) q.row[d] = *(const float4*)(rows + (size_t)(e0 + (unsigned)min(16 * d + c, s.D - 1)) * 16u);
}

// Powers N0 + 1 .. N1 of one k-step: A the pixel factors U^n (advanced), C the
// coefficients of the lane's line at depths 16 d + c.
template <int N0, int N1, int NPT>
__device__ __forceinline__ void far_powers(f32x4 (*acc)[FAR_NDT], float* A, const float* u, const bool* live,
                                           const FarStep& q, float x0, bool zone, int ndt) {
    float P[NPT][N1 - N0];
#pragma unroll
    for (int t = 0; t < NPT; ++t)
#pragma unroll
        for (int n = 0; n < N1 - N0; ++n) {
            P[t][n] = A[t];
            A[t] *= u[t];
        }
#pragma unroll
    for (int d = 0; d < FAR_NDT; ++d)
        if (d < ndt) {
            const float sx = q.row[d].x * x0;
            const float W = zone ? __builtin_amdgcn_rcpf(sx * sx) : 0.0f;
            float lead = zone ? q.row[d].w * W * kInvSqrtPiF : 0.0f, C[N1 - N0];
#pragma unroll
            for (int n = 0; n < N0; ++n) lead *= W;
            far_poly<N0, N1>(PZ_FAR_H, zone ? q.row[d].y : 0.0f, W, lead, C);
#pragma unroll
            for (int t = 0; t < NPT; ++t)
                if (live[t]) {
#pragma unroll
                    for (int n = 0; n < N1 - N0; ++n)
                        acc[t][d] = __builtin_amdgcn_mfma_f32_16x16x4f32(P[t][n], C[n], acc[t][d], 0, 0, 0);
                }
        }
}

template <int NPT>
__device__ __forceinline__ void dev_opacity_far(const StarDev& s, int tile, FarLds<NPT>& lds) {
    const int lane = threadIdx.x % WAVE, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int nw = blockDim.x / WAVE;                     // far_waves<NPT>()
    const int c = lane % 16, r = lane / 16;
    constexpr int T32 = NPT / 2;                          // tiles of the line lists
    const int p0 = tile * (16 * NPT);
    const int l0 = s.t32_first[tile * T32], l1 = s.t32_last[min(tile * T32 + T32 - 1, s.n_t32 - 1)];
    const int D = s.D, ndt = (D + 15) / 16;
    f32x4 acc[NPT][FAR_NDT];
#pragma unroll
    for (int t = 0; t < NPT; ++t)
#pragma unroll
        for (int d = 0; d < FAR_NDT; ++d) acc[t][d] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const char* rows = scalar_base(s.lp + (size_t)l0 * D);
    FarStep q, next;
    int b = l0 + 4 * wave;
    if (b < l1) far_load(s, rows, l0, l1, b, r, c, ndt, next);
    for (; b < l1; b += 4 * nw) {
        q = next;
        if (b + 4 * nw < l1) far_load(s, rows, l0, l1, b + 4 * nw, r, c, ndt, next);
        float u[NPT], A[NPT];
        bool live[NPT];
        float um = 0.0f;
#pragma unroll
        for (int t = 0; t < NPT; ++t) {
            const int i = p0 + 16 * t + c;
            const float x = detuning(i - q.ic, q.dl, s.h_hi, s.h_lo);
            const float w = q.xf * __builtin_amdgcn_rcpf(x);
            u[t] = i >= q.lo && i <= q.hi && in_far_zone(x, q.xf) ? w * w : 0.0f;
            live[t] = wave_any(u[t] > 0.0f);
            um = fmaxf(um, u[t]);
            A[t] = u[t];
        }
        if (!wave_any(um > 0.0f)) continue;
        const bool zone = q.xf >= 0.0f && q.xf < INFINITY;
        far_powers<0, 2, NPT>(acc, A, u, live, q, q.xf, zone, ndt);
        if (!wave_any(um > kFarU2)) continue;
        far_powers<2, 3, NPT>(acc, A, u, live, q, q.xf, zone, ndt);
        if (!wave_any(um > kFarU3)) continue;
        far_powers<3, 4, NPT>(acc, A, u, live, q, q.xf, zone, ndt);
        if (!wave_any(um > kFarU4)) continue;
        far_powers<4, PZ_FAR_N, NPT>(acc, A, u, live, q, q.xf, zone, ndt);
    }
    // Add the wavefronts' sums: the upper half of them into the lower half
    // through LDS, a 16-pixel block at a time, until one is left.
    for (int m = nw / 2; m > 0; m /= 2) {
#pragma unroll
        for (int t = 0; t < NPT; ++t) {
            if (wave >= m && wave < 2 * m)
#pragma unroll
                for (int d = 0; d < FAR_NDT; ++d)
                    if (d < ndt) lds.part[wave - m][d][lane] = acc[t][d];
            __syncthreads();
            if (wave < m)
#pragma unroll
                for (int d = 0; d < FAR_NDT; ++d)
                    if (d < ndt) acc[t][d] += lds.part[wave][d][lane];
            __syncthreads();
        }
    }
    if (wave == 0)
#pragma unroll
        for (int t = 0; t < NPT; ++t)
#pragma unroll
            for (int d = 0; d < FAR_NDT; ++d) {
                const int j = 16 * d + c;
                // lane (r, c) holds pixels 4 r .. 4 r + 3 of the block at depth c
                if (d < ndt && j < D) *(f32x4*)(s.kappa + (size_t)j * s.Npad + p0 + 16 * t + 4 * r) = acc[t][d];
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

template <bool FULL, int NG, bool CT>
__device__ __forceinline__ void near_sums(float* acc, const float4* p, const float* v, const float* zm,
                                          const float4* near_tab) {
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const float a = near_KH_acc<FULL>(acc[g], p[g].y, p[g].z, p[g].w, v[g], near_tab);
        acc[g] = !CT || fmaf(v[g], v[g], p[g].y) <= zm[g] ? a : acc[g];
    }
}

template <int NG, bool CT>
__device__ __forceinline__ void near_line(float* acc, const float4* p, const float* zm, float x, bool safe,
                                          const float4* near_tab, const float4* pw) {
    float v[NG], amax = p[0].y, smax = fabsf(p[0].x);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        v[g] = x * p[g].x;
        if (g > 0) {
            amax = fmaxf(amax, p[g].y);
            smax = fmaxf(smax, fabsf(p[g].x));
        }
    }
    if (!safe && wave_all(amax <= PZ_VOIGT_A2_SMALL) && wave_all(smax * fabsf(x) < PZ_NEAR_V)) {
        if (wave_any(amax > PZ_VOIGT_A2_TINY))
            near_sums<true, NG, CT>(acc, p, v, zm, near_tab);
        else
            near_sums<false, NG, CT>(acc, p, v, zm, near_tab);
        return;
    }
    float z2[NG], zmin = INFINITY;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        z2[g] = fmaf(v[g], v[g], p[g].y);
        zmin = fminf(zmin, z2[g]);
    }
    if (!safe && wave_all(zmin >= PZ_VOIGT_WING_R2)) {
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
    bool some = false;                                    // a line in reach of the wavefront's pixels
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
        // (a line between two pixels can have none in its window: lo > hi)
        unsigned long long m = __builtin_amdgcn_ballot_w64(b + lane < l1 && lo <= hi && lo <= p0 + 7 && hi >= p0);
        const unsigned long long wide = __builtin_amdgcn_ballot_w64(xf < 0.0f);
        some = some || m;
        while (m) {
            const int k = __builtin_ctzll(m);
            m &= m - 1;
            const float x = detuning(i - __builtin_amdgcn_readlane(ic, k), __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dl), k)),
                                     s.h_hi, s.h_lo);
            const float rc = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(reach), k));
            const int klo = __builtin_amdgcn_readlane(lo, k), kn = __builtin_amdgcn_readlane(hi, k) - klo;
            const bool in = ((unsigned)(i - klo) <= (unsigned)kn) & (fabsf(x) < rc);
            if (in) {
                const size_t e = (size_t)(b + k) * D;
                const char* row = (const char*)(s.lp + e);
                float4 p[NG];
                float zm[NG];
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    unsigned o = off[g];
                    asm volatile("" : "+v"(o));           // keeps the 32-bit offset on a scalar base
                    p[g] = *(const float4*)(row + o);
                    zm[g] = CT ? *(const float*)((const char*)(s.zmax + e) + o / 4u) : 0.0f;
                }
                near_line<NG, CT>(acc, p, zm, x, (wide >> k) & 1, near_tab, pw);
            }
        }
    }
    if (some && i < s.N) {
#pragma unroll
        for (int g = 0; g < NG; ++g)
            if (j0 + 8 * g < D) s.kappa[(size_t)(j0 + 8 * g) * s.Npad + i] += acc[g];
    }
}

}  // namespace pz
