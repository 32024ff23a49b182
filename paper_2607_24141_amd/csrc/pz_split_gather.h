// Line-parallel adjoint of the split sums (pz_split.h): per line, the sums over
// its window of g K H, g K a dH/da and g (-K X d ln dnu_D / d xi), g =
// dL/dkappa.  The far zone is a matrix product (here), the near zone the direct
// gather of pz_stages.h within the zone limit, whose results it adds.
//
// Both gathers so take one form of a dH/da in the core.  Another one (from a
// table of Dawson's integral, nearer to float64) differs by 1e-6 of the terms
// between which a dH/da is formed; in saturated spectra a line's damping
// gradient is what is left of terms that cancel to 1e-3, and single entries
// then moved by up to 4.4e-3 of max(rms, |entry|) against the direct gather
// (1500-1700 nm with 200,000 lines, 61 seeds; now 3e-4, the opacity's rounding).
#pragma once

namespace pz {

// The five sums of a line: gf, damping (or radiative), xi, Stark, van der Waals.
struct LineSums {
    float gf, d, xi, ds, dw;
};

// Shares of the damping width by family at depth j (radiative, Stark, van der Waals).
__device__ __forceinline__ float3 family_shares(const StarDev& s, const double4& c, int j) {
    const float gr = (float)c.y, Gs = (float)c.z * (float)s.ne[j], Gw = (float)c.w * (float)s.npert[j];
    const float inv = 1.0f / (gr + Gs + Gw);
    return make_float3(gr * inv, Gs * inv, Gw * inv);
}

// ------------------------------------------------------------------ far zone
// T_n[line][depth] = sum_pixels U^n g, U = (xfar/x)^2 in the line's far zone
// and 0 elsewhere: for each power a (line x pixel) by (pixel x depth) product.
// K H, K a dH/da and K X are combinations of the same T_n (far_poly), so the
// window is passed once for all three.  One wavefront per 16 lines: the
// sorted lines' windows nearly coincide, and a chunk of 16 pixels is four
// k-steps (lane (r, c) = (lane / 16, lane % 16): line c and pixels 4 r + t, t =
// 0..3, of the chunk; B is a float4 of dL/dkappa at depth c).  Chunks with no
// far pixel are skipped.
// Powers whose terms cannot reach 1e-6 of X at a chunk's nearest pixel are left
// out: X has lost its leading order and needs one power more than H does (H and
// a dH/da lose less than 2e-9).  Measured in units of x0, where v >= 5.5 and
// a <= 0.2 v: n <= 5 from v = 16, n <= 4 from 25, n <= 3 from 74.  With all six
// X is within 1.8e-5 (at v = 5.5; the direct gather's far-wing series: 9e-5).
// Two wavefronts share the lines and split the depth tiles (three and two), so
// the powers' sums fit beside a chunk's operands and the next chunk's loads;
// the second hands its line sums over through LDS.
static constexpr float kGFarU5 = 0.12f;                   // (5.5/16)^2
static constexpr float kGFarU4 = 0.05f;                   // (5.5/25)^2
static constexpr float kGFarU3 = 0.0055f;                 // (5.5/74)^2
static constexpr int GFAR_LINES = 16;
static constexpr int GFAR_NDT = 3;                        // depth tiles per wavefront
static_assert(2 * GFAR_NDT >= FAR_NDT, "two wavefronts cover the depths");

// Powers N0 + 1 .. N1 of one chunk.
template <int N0, int N1>
__device__ __forceinline__ void gather_powers(f32x4 (*T)[GFAR_NDT], float* A, const float* u, const f32x4* g, int ndt) {
#pragma unroll
    for (int n = N0; n < N1; ++n) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int d = 0; d < GFAR_NDT; ++d)
                if (d < ndt) T[n][d] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[t], g[d][t], T[n][d], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < 4; ++t) A[t] *= u[t];
    }
}

// Sums the far zone of lines base .. base + 15 into gline, unscaled; called by
// two wavefronts (half = 0, 1) of a workgroup, which it synchronises.  hand:
// the pair's LDS.
template <bool FAM>
__device__ __forceinline__ void dev_gather_far(const StarDev& s, int base, int half, LineSums* hand) {
    const int lane = threadIdx.x % WAVE, c = lane % 16, r = lane / 16;
    const int D = s.D, d0 = half * GFAR_NDT, ndt = min((D + 15) / 16 - d0, GFAR_NDT);   // may be <= 0
    const int l = min(base + c, s.L - 1);
    const float xf = base + c < s.L ? s.xfar[l] : -1.0f;
    const bool zone = xf >= 0.0f && xf < INFINITY && ndt > 0;
    const int ic = s.ln.ic[l];
    const float dl = s.ln.delta[l];
    const int lo = zone ? s.ln.ilo[l] : s.N, hi = zone ? s.ln.ihi[l] : -1;
    int i0 = lo, i1 = hi;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {                     // over the 16 lines (any 16 neighbouring lanes)
        i0 = min(i0, __shfl_xor(i0, o, WAVE));
        i1 = max(i1, __shfl_xor(i1, o, WAVE));
    }
    i0 = __builtin_amdgcn_readfirstlane(i0) & ~15;
    i1 = __builtin_amdgcn_readfirstlane(i1);
    f32x4 T[PZ_FAR_N][GFAR_NDT];
#pragma unroll
    for (int n = 0; n < PZ_FAR_N; ++n)
#pragma unroll
        for (int d = 0; d < GFAR_NDT; ++d) T[n][d] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const float* gp[GFAR_NDT];
#pragma unroll
    for (int d = 0; d < GFAR_NDT; ++d) gp[d] = s.gk + (size_t)min(16 * (d0 + d) + c, D - 1) * s.Npad + 4 * r;
    bool spoilt = false;                                  // a non-finite g inside the line's far zone
    f32x4 next[GFAR_NDT];
#pragma unroll
    for (int d = 0; d < GFAR_NDT; ++d) next[d] = i0 <= i1 ? *(const f32x4*)(gp[d] + i0) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    for (int i = i0, nx; i <= i1; i = nx) {
        // the next chunk that a window reaches: the sorted lines' windows begin and end in order, so the
        // first line that goes on beyond this chunk has it (none: the end)
        const unsigned on = (unsigned)__builtin_amdgcn_ballot_w64(hi >= i + 16) & 0xffffu;
        nx = on ? max(i + 16, __builtin_amdgcn_readlane(lo, __builtin_ctz(on)) & ~15) : i1 + 1;
        f32x4 g[GFAR_NDT];
        f32x4 fin = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int d = 0; d < GFAR_NDT; ++d) {
            g[d] = next[d];
            fin += g[d] * 0.0f;
        }
        if (nx <= i1)
#pragma unroll
            for (int d = 0; d < GFAR_NDT; ++d) next[d] = *(const f32x4*)(gp[d] + nx);
        float u[4], A[4], um = 0.0f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int p = i + 4 * r + t;
            const float x = detuning(p - ic, dl, s.h_hi, s.h_lo);
            const float q = xf * __builtin_amdgcn_rcpf(x);
            u[t] = p >= lo && p <= hi && in_far_zone(x, xf) ? q * q : 0.0f;
            um = fmaxf(um, u[t]);
            A[t] = u[t];
        }
        if (!wave_any(um > 0.0f)) continue;
        if (wave_any(!(fin.x + fin.y + fin.z + fin.w == 0.0f))) {
            // a non-finite g reaches the lines whose far zone holds its pixel and no others
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const unsigned long long b = __builtin_amdgcn_ballot_w64(!(fin[t] == 0.0f));
                if ((b >> (16 * r)) & 0xffffull) spoilt = spoilt || u[t] > 0.0f;
            }
#pragma unroll
            for (int d = 0; d < GFAR_NDT; ++d)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (!(fabsf(g[d][t]) < INFINITY)) g[d][t] = 0.0f;
        }
        gather_powers<0, 3>(T, A, u, g, ndt);
        if (!wave_any(um > kGFarU3)) continue;
        gather_powers<3, 4>(T, A, u, g, ndt);
        if (!wave_any(um > kGFarU4)) continue;
        gather_powers<4, 5>(T, A, u, g, ndt);
        if (!wave_any(um > kGFarU5)) continue;
        gather_powers<5, PZ_FAR_N>(T, A, u, g, ndt);
    }
    // lane (r, c) holds lines base + 4 r + q, q = 0..3, at depths 16 (d0 + d) + c
    const float xi_f = s.xi[0] * (float)(1.0e10 / (C_LIGHT * C_LIGHT));
    const unsigned long long sp = __builtin_amdgcn_ballot_w64(spoilt);   // line k's lanes: c = k - base
    LineSums out[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int kl = min(base + 4 * r + q, s.L - 1);
        const float xk = s.xfar[kl];
        const bool zk = xk >= 0.0f && xk < INFINITY;
        LineSums o = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        const double4 lc = FAM ? s.lc[kl] : make_double4(0.0, 0.0, 0.0, 0.0);
#pragma unroll
        for (int d = 0; d < GFAR_NDT; ++d) {
            const int j = 16 * (d0 + d) + c;
            if (j >= D || !zk) continue;
            const float4 p = s.lp[(size_t)kl * D + j];
            const float sx = p.x * xk, W = __builtin_amdgcn_rcpf(sx * sx);
            float C[PZ_FAR_N], h = 0.0f, a = 0.0f, x = 0.0f;
            const float lead = p.w * W * kInvSqrtPiF;
            far_poly<0, PZ_FAR_N>(PZ_FAR_H, p.y, W, lead, C);
#pragma unroll
            for (int n = 0; n < PZ_FAR_N; ++n) h = fmaf(C[n], T[n][d][q], h);
            far_poly<0, PZ_FAR_N>(PZ_FAR_A, p.y, W, lead, C);
#pragma unroll
            for (int n = 0; n < PZ_FAR_N; ++n) a = fmaf(C[n], T[n][d][q], a);
            far_poly<0, PZ_FAR_N - 1>(PZ_FAR_X, p.y, W, lead * W, C);
#pragma unroll
            for (int n = 0; n < PZ_FAR_N - 1; ++n) x = fmaf(C[n], T[n + 1][d][q], x);
            o.gf += h;
            o.xi = fmaf(x, -xi_f * p.x * p.x, o.xi);
            if (FAM) {
                const float3 f = family_shares(s, lc, j);
                o.d = fmaf(a, f.x, o.d);
                o.ds = fmaf(a, f.y, o.ds);
                o.dw = fmaf(a, f.z, o.dw);
            } else {
                o.d += a;
            }
        }
#pragma unroll
        for (int w = 8; w > 0; w >>= 1) {
            o.gf += __shfl_xor(o.gf, w, WAVE);
            o.d += __shfl_xor(o.d, w, WAVE);
            o.xi += __shfl_xor(o.xi, w, WAVE);
            if (FAM) {
                o.ds += __shfl_xor(o.ds, w, WAVE);
                o.dw += __shfl_xor(o.dw, w, WAVE);
            }
        }
        if (((sp | (sp >> 16) | (sp >> 32) | (sp >> 48)) >> (4 * r + q)) & 1ull) {
            const float nan = __builtin_nanf("");
            o = {nan, nan, nan, nan, nan};
        }
        out[q] = o;
    }
    if (half == 1 && c == 0)
#pragma unroll
        for (int q = 0; q < 4; ++q) hand[4 * r + q] = out[q];
    __syncthreads();
    if (half == 0 && c == 0)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = base + 4 * r + q;
            if (k >= s.L) break;
            const LineSums h = hand[4 * r + q];
            s.gline[k] = out[q].gf + h.gf;
            s.gline[s.L + k] = out[q].d + h.d;
            s.gline[2 * s.L + k] = out[q].xi + h.xi;
            if (FAM) {
                s.gline[3 * s.L + k] = out[q].ds + h.ds;
                s.gline[4 * s.L + k] = out[q].dw + h.dw;
            }
        }
}

}  // namespace pz
