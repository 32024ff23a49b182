// Line-parallel adjoint of the split sums (pz_split.h): per line, the sums over
// its window of g K H, g K a dH/da and g (-K X d ln dnu_D / d xi), g =
// dL/dkappa, the far zone as a matrix product and the near zone directly.
// Included by pz_stages.h, whose wave_sum and far_series it uses.
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
// far pixel are skipped; powers are dropped as in dev_opacity_far.
// Two wavefronts share the lines and split the depth tiles (three and two), so
// the powers' sums fit beside a chunk's operands and the next chunk's loads;
// the second hands its line sums over through LDS.
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
    for (int i = i0; i <= i1; i += 16) {
        f32x4 g[GFAR_NDT];
        f32x4 fin = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int d = 0; d < GFAR_NDT; ++d) {
            g[d] = next[d];
            fin += g[d] * 0.0f;
        }
        if (i + 16 <= i1)
#pragma unroll
            for (int d = 0; d < GFAR_NDT; ++d) next[d] = *(const f32x4*)(gp[d] + i + 16);
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
        gather_powers<0, 2>(T, A, u, g, ndt);
        if (!wave_any(um > kFarU2)) continue;
        gather_powers<2, 3>(T, A, u, g, ndt);
        if (!wave_any(um > kFarU3)) continue;
        gather_powers<3, 4>(T, A, u, g, ndt);
        if (!wave_any(um > kFarU4)) continue;
        gather_powers<4, PZ_FAR_N>(T, A, u, g, ndt);
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

// ----------------------------------------------------------------- near zone
// One wavefront per line, lanes (pixel p, depth q) = (lane % 8, lane / 8): the
// near zone is passed 32 pixels at a time (8 per step, up to four steps held
// in registers), depth groups of 8 outside, so a parameter row is read once
// per 32 pixels and the steps are independent straight-line chains.  Pixels
// outside the zone enter with x = 0 and g = 0.
static constexpr int GNEAR_STEPS = 4;

template <bool FULL>
__device__ __forceinline__ void near_terms(const float4& q, const float* x, const float* g, int ns, const float4* near_tab,
                                           float& sgf, float& sd, float& sx) {
#pragma unroll
    for (int t = 0; t < GNEAR_STEPS; ++t)
        if (t < ns) {
            float h, a, X;
            near_KHD<FULL>(q.y, q.z, q.w, x[t] * q.x, near_tab, h, a, X);
            sgf = fmaf(g[t], h, sgf);
            sd = fmaf(g[t], a, sd);
            sx = fmaf(g[t], X, sx);
        }
}

template <bool CT, bool FAM>
__device__ __forceinline__ void dev_gather_near(const StarDev& s, int l, int lane, const float4* near_tab,
                                                const float4* pw) {
    const int D = s.D, px = lane % 8, dg = lane / 8;
    const float xf = s.xfar[l], dl = s.ln.delta[l];
    const int ic = s.ln.ic[l];
    int lo = s.ln.ilo[l], hi = s.ln.ihi[l];
    float reach = near_reach(xf);
    if (CT) reach = fminf(reach, s.xlim[l] * (1.0f + 1e-5f));
    // pixels with |x| < reach lie within (reach + reach^2) / h + 1/2 of the anchor
    const float wpx = fmaf(reach, reach, reach) / s.h_hi + 2.0f;
    if (reach < 0.5f && wpx < 1.0e6f) {
        lo = max(lo, ic - (int)wpx);
        hi = min(hi, ic + (int)wpx);
    }
    const float xi_f = s.xi[0] * (float)(1.0e10 / (C_LIGHT * C_LIGHT));
    const double4 lc = FAM ? s.lc[l] : make_double4(0.0, 0.0, 0.0, 0.0);
    const float4* row = s.lp + (size_t)l * D;
    const float* zrow = CT ? s.zmax + (size_t)l * D : nullptr;
    LineSums o = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    for (int p0 = lo; p0 <= hi; p0 += 8 * GNEAR_STEPS) {
        const int ns = min((hi - p0 + 8) / 8, GNEAR_STEPS);
        float x[GNEAR_STEPS], xm = 0.0f;
        bool in[GNEAR_STEPS];
#pragma unroll
        for (int t = 0; t < GNEAR_STEPS; ++t) {
            const int i = p0 + 8 * t + px;
            x[t] = detuning(i - ic, dl, s.h_hi, s.h_lo);
            in[t] = i <= hi && fabsf(x[t]) < reach;
            x[t] = in[t] ? x[t] : 0.0f;
            xm = fmaxf(xm, fabsf(x[t]));
        }
        const float* gp = s.gk + p0 + px;
#pragma unroll 1
        for (int j0 = 0; j0 < D; j0 += 8) {
            const int j = min(j0 + dg, D - 1);
            const bool jin = j0 + dg < D;
            const float4 q = row[j];
            const float zm = CT ? zrow[j] : 0.0f;
            const float* g = gp + (size_t)j * s.Npad;
            float gj[GNEAR_STEPS];
#pragma unroll
            for (int t = 0; t < GNEAR_STEPS; ++t) {
                bool take = in[t] && jin;
                if (CT) {
                    const float v = x[t] * q.x;
                    take = take && fmaf(v, v, q.y) <= zm;
                }
                gj[t] = take ? g[8 * t] : 0.0f;
            }
            float sgf = 0.0f, sd = 0.0f, sx = 0.0f;
            if (wave_all(q.y <= PZ_VOIGT_A2_SMALL) && wave_all(fabsf(q.x) * xm < PZ_NEAR_V)) {
                if (wave_any(q.y > PZ_VOIGT_A2_TINY))
                    near_terms<true>(q, x, gj, ns, near_tab, sgf, sd, sx);
                else
                    near_terms<false>(q, x, gj, ns, near_tab, sgf, sd, sx);
            } else {
                float z2[GNEAR_STEPS], zmin = INFINITY;
#pragma unroll
                for (int t = 0; t < GNEAR_STEPS; ++t) {
                    const float v = x[t] * q.x;
                    z2[t] = gj[t] != 0.0f ? fmaf(v, v, q.y) : kFarZ2;      // also takes a NaN g
                    zmin = fminf(zmin, z2[t]);
                }
                if (wave_all(zmin >= kFarZ2) && wave_all(q.y <= kFarB)) {
#pragma unroll
                    for (int t = 0; t < GNEAR_STEPS; ++t)
                        if (t < ns) {
                            float r, th, ta, tx;
                            far_series(q.y, z2[t], r, th, ta, tx);
                            const float w = (gj[t] * r) * (q.w * kInvSqrtPiF);
                            sgf = fmaf(w, th, sgf);
                            sd = fmaf(w, ta, sd);
                            sx = fmaf(w, tx * r, sx);
                        }
                } else {
#pragma unroll 1
                    for (int t = 0; t < ns; ++t) {
                        float xt = x[0], gt = gj[0];
#pragma unroll
                        for (int k = 1; k < GNEAR_STEPS; ++k)
                            if (t == k) {
                                xt = x[k];
                                gt = gj[k];
                            }
                        if (gt != 0.0f) {
                            const float v = xt * q.x;
                            float th, ta, tx;
                            voigt_KHD(q.y, q.z, q.w, v, v * v, pw, th, ta, tx);
                            sgf = fmaf(gt, th, sgf);
                            sd = fmaf(gt, ta, sd);
                            sx = fmaf(gt, tx, sx);
                        }
                    }
                }
            }
            o.gf += sgf;
            o.xi = fmaf(sx, -xi_f * q.x * q.x, o.xi);
            if (FAM) {
                const float3 f = family_shares(s, lc, j);
                o.d = fmaf(sd, f.x, o.d);
                o.ds = fmaf(sd, f.y, o.ds);
                o.dw = fmaf(sd, f.z, o.dw);
            } else {
                o.d += sd;
            }
        }
    }
    o.gf = wave_sum(o.gf);
    o.d = wave_sum(o.d);
    o.xi = wave_sum(o.xi);
    if (FAM) {
        o.ds = wave_sum(o.ds);
        o.dw = wave_sum(o.dw);
    }
    if (lane == 0) {                                      // the far zone's sums are in gline
        s.gline[l] = (float)LN10 * (s.gline[l] + o.gf);
        s.gline[s.L + l] = (float)LN10 * (s.gline[s.L + l] + o.d);
        s.gline[2 * s.L + l] += o.xi;
        if (FAM) {
            s.gline[3 * s.L + l] = (float)LN10 * (s.gline[3 * s.L + l] + o.ds);
            s.gline[4 * s.L + l] = (float)LN10 * (s.gline[4 * s.L + l] + o.dw);
        }
    }
}

__device__ __forceinline__ void dev_gather_split(const StarDev& s, int l, int lane, const float4* near_tab,
                                                 const float4* pw) {
    if (l >= s.L) return;
    if (s.fam) {
        if (s.center)
            dev_gather_near<true, true>(s, l, lane, near_tab, pw);
        else
            dev_gather_near<false, true>(s, l, lane, near_tab, pw);
    } else {
        if (s.center)
            dev_gather_near<true, false>(s, l, lane, near_tab, pw);
        else
            dev_gather_near<false, false>(s, l, lane, near_tab, pw);
    }
}

}  // namespace pz
