// The transfer by one thread per pixel: a single walk along depth, which the
// row forms of pz_stages.h split over lanes.  The walk has no scans, idle
// lanes or padding of the depths, so it has the higher rate; a chip it does not
// fill waits for its serial chain instead.  columns_rule chooses.
// Included by pz_stages.h.
#pragma once

#include <algorithm>
#include <cmath>

namespace pz {

// The rays of the formal solution, from the surface down.
struct Ray3 {
    float F[3], A[3];
    __device__ void top(float S0, float S1, float t0, float t1) {
        const float S_top = S0 - t0 * (S1 - S0) / (t1 - t0);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const ExpTerms et = exp_terms(t0 * c_inv_mu[k]);
            F[k] = fmaf(S_top, et.om, (S0 - S_top) * et.lw);
            A[k] = et.e;
        }
    }
    __device__ void seg(float Sa, float Sb, float ta, float tb) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const ExpTerms et = exp_terms((tb - ta) * c_inv_mu[k]);
            const float c = fmaf(Sa, et.om, (Sb - Sa) * et.lw);
            F[k] = fmaf(A[k], c, F[k]);
            A[k] *= et.e;
        }
    }
    __device__ float bottom(float Sa, float Sb, float ta, float tb) {
        const float grad = (Sb - Sa) / (tb - ta);
        float out = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float ID = fmaf(c_mu[k], grad, Sb);
            out = fmaf(c_wmu[k], fmaf(A[k], ID, F[k]), out);
        }
        return out;
    }
};

// Copies pixel i's column into col (stride WAVE): sixteen loads in flight per
// wait instead of one per depth step.  Only the calling thread reads it back.
template <class T>
__device__ __forceinline__ void stage_kappa_column(const StarDev& s, int i, T* col) {
    const float* kl = s.kappa + i;
    const int D = s.D;
    for (int j0 = 0; j0 < D; j0 += 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = kl[(size_t)min(j0 + u, D - 1) * s.Npad];
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (j0 + u < D) col[(j0 + u) * WAVE] = (T)v[u];
    }
}

// Gauss-3 flux of pixel i on the total branch (TOT; col: its staged column) or
// the continuum branch, float32: the same bits as dev_flux_block.
template <bool TOT>
__device__ __forceinline__ void dev_flux_column(const StarDev& s, int i, const float* col) {
    if (i >= s.N) return;
    const PixelSetup p = pixel_setup(s, i);
    const int D = s.D;
    auto chi = [&](int j) { return TOT ? p.kc + col[j * WAVE] : p.kc; };
    float mb = (float)s.m[1], Sa = planck(p, (float)(1.0 / s.T[0])), Sb = planck(p, (float)(1.0 / s.T[1]));
    const float m0 = (float)s.m[0], chi0 = chi(0);
    float chib = chi(1), ta = chi0 * m0, tb = fmaf(TOT ? 0.5f * (chi0 + chib) : p.kc, mb - m0, ta);
    Ray3 r;
    r.top(Sa, Sb, ta, tb);
    r.seg(Sa, Sb, ta, tb);
    for (int j = 2; j < D; ++j) {
        const float mj = (float)s.m[j], chij = chi(j);
        Sa = Sb;
        Sb = planck(p, (float)(1.0 / s.T[j]));
        ta = tb;
        tb = fmaf(TOT ? 0.5f * (chib + chij) : p.kc, mj - mb, ta);
        chib = chij;
        mb = mj;
        r.seg(Sa, Sb, ta, tb);
    }
    (TOT ? s.F : s.Fc)[i] = r.bottom(Sa, Sb, ta, tb);
}

struct RayE2 {
    double F, E3a, E4a;
    __device__ void start() {
        F = 0.0;
        E3a = 0.5;            // E3(0)
        E4a = 1.0 / 3.0;      // E4(0)
    }
    __device__ void seg(double Sa, double Sb, double ta, double tb) {
        double E3b, E4b;
        expint34(tb, E3b, E4b);
        const double sl = (Sb - Sa) / (tb - ta);
        F += Sa * (E3a - E3b) + sl * (E4a - E4b - (tb - ta) * E3b);
        E3a = E3b;
        E4a = E4b;
    }
    __device__ double bottom(double Sa, double Sb, double ta, double tb) const {
        const double sD = (Sb - Sa) / (tb - ta);
        return 2.0 * PI * (F + Sb * E3a + sD * E4a);
    }
};

// E2 flux of pixel i on the total branch (TOT; col: its staged column) or the
// continuum branch, float64.
template <bool TOT>
__device__ __forceinline__ void dev_flux_e2_column(const StarDev& s, int i, const float* col) {
    if (i >= s.N) return;
    const PixelSetup64 p = pixel_setup64(s, i);
    const int D = s.D;
    auto chi = [&](int j) { return TOT ? p.kc + (double)col[j * WAVE] : p.kc; };
    double mb = s.m[1], Sa = p.planck(s.T[0]), Sb = p.planck(s.T[1]);
    const double chi0 = chi(0);
    double chib = chi(1), ta = chi0 * s.m[0], tb = ta + 0.5 * (chi0 + chib) * (mb - s.m[0]);
    RayE2 r;
    r.start();
    r.seg(Sa - ta * (Sb - Sa) / (tb - ta), Sa, 0.0, ta);  // from tau = 0 with the first segment's slope
    r.seg(Sa, Sb, ta, tb);
    for (int j = 2; j < D; ++j) {
        const double mj = s.m[j], chij = chi(j);
        Sa = Sb;
        Sb = p.planck(s.T[j]);
        ta = tb;
        tb = ta + 0.5 * (chib + chij) * (mj - mb);
        chib = chij;
        mb = mj;
        r.seg(Sa, Sb, ta, tb);
    }
    (TOT ? s.F : s.Fc)[i] = (float)r.bottom(Sa, Sb, ta, tb);
}

// The reverse of the E2 flux as in dev_reverse_e2_row.
// col: pixel i's float64 LDS column (stride WAVE), holding kappa_line on
// entry and dL/dtau after (each depth written once, as in dev_reverse_column).
__device__ __forceinline__ void dev_reverse_e2_column(const StarDev& s, int i, double* col) {
    if (i >= s.N) return;
    const int D = s.D;
    const double G = 2.0 * PI * (double)s.dLdF[i];
    const PixelSetup64 p = pixel_setup64(s, i);
    const double kc = p.kc;
    const double S0 = p.planck(s.T[0]), S1 = p.planck(s.T[1]);
    const double chi0 = kc + col[0], chi1 = kc + col[WAVE];
    const double t0 = chi0 * s.m[0];
    const double t1 = t0 + 0.5 * (chi0 + chi1) * (s.m[1] - s.m[0]);
    const double d01 = t1 - t0, sig = (S1 - S0) / d01;
    double E3a, E4a;
    expint34(t0, E3a, E4a);
    double g0, g1;                                     // top-slab terms of dL/dtau_0, dL/dtau_1
    {
        const double dE3 = 0.5 - E3a;                       // E3(0) - E3(tau_0)
        const double P0 = 1.0 / 3.0 - E4a - t0 * E3a;        // E4(0) - E4(tau_0) - tau_0 E3(tau_0)
        g0 = G * (dE3 * (-sig - t0 * sig / d01) + P0 * sig / d01);
        g1 = G * (dE3 * (t0 * sig / d01) - P0 * sig / d01);
    }
    double Sa = S0, Sb = S1, ta = t0, tb = t1, chib = chi1, mb = s.m[1];
    double pend = g1, last = 0.0;                      // pend: what depth j + 1 already holds
    for (int j = 0; j < D - 1; ++j) {
        if (j > 0) {
            const double mj = s.m[j + 1];
            const double chij = kc + col[(j + 1) * WAVE];
            Sa = Sb;
            ta = tb;
            Sb = p.planck(s.T[j + 1]);
            tb = ta + 0.5 * (chib + chij) * (mj - mb);
            chib = chij;
            mb = mj;
        }
        double E3b, E4b;
        expint34(tb, E3b, E4b);
        const double dt = tb - ta, sl = (Sb - Sa) / dt;
        const double P = E4a - E4b - dt * E3b;
        const double gj = (j == 0 ? g0 : pend) + G * (sl * (E3b - E3a) + P * sl / dt);
        if (j < D - 2)
            col[j * WAVE] = gj;
        else
            last = gj;
        pend = (j == 0 ? g1 : 0.0) + G * (-P * sl / dt);
        E3a = E3b;
        E4a = E4b;
    }
    {
        const double dt = tb - ta, sD = (Sb - Sa) / dt;
        col[(D - 2) * WAVE] = last + G * (E4a * sD / dt);
        col[(D - 1) * WAVE] = pend + G * (-sD * E3a - E4a * sD / dt);
    }
    double suffix = 0.0, gnext = 0.0;
    float* out = s.gk + i;
    const size_t st = s.Npad;
    for (int j = D - 1; j >= 0; --j) {
        suffix += col[j * WAVE];
        double g = (j == D - 1) ? 0.0 : 0.5 * (s.m[j + 1] - s.m[j]) * gnext;
        g += (j == 0) ? s.m[0] * suffix : 0.5 * (s.m[j] - s.m[j - 1]) * suffix;
        out[(size_t)j * st] = (float)g;
        gnext = suffix;
    }
}

// Pixel i's column of a workgroup of WAVE pixels: col[j * WAVE], float64 in
// LDS.  On entry it holds kappa_line[j][i]; the scan overwrites slot j with
// dL/dtau_j once kappa_line[j] has been read (each slot is written once: the
// term a segment adds to the next depth is carried in a register), then the
// trapezoid adjoint runs up from the bottom.
__device__ __forceinline__ void dev_reverse_column(const StarDev& s, int i, double* col) {
    if (i >= s.N) return;
    const int D = s.D;
    const double G = s.dLdF[i];
    const double mu[3] = {kMu0, kMu1, kMu2};
    const double wmu[3] = {2.0 * PI * 5.0 / 18.0 * kMu0, 2.0 * PI * 8.0 / 18.0 * kMu1, 2.0 * PI * 5.0 / 18.0 * kMu2};
    const PixelSetup64 p = pixel_setup64(s, i);
    const double kc = p.kc;
    // surface quantities
    const double m0 = s.m[0], m1 = s.m[1];
    const double S0 = p.planck(s.T[0]);
    const double S1 = p.planck(s.T[1]);
    const double chi0 = kc + col[0], chi1 = kc + col[WAVE];
    const double t0 = chi0 * m0;
    const double t1 = t0 + 0.5 * (chi0 + chi1) * (m1 - m0);
    const double dt01 = t1 - t0;
    const double sig = (S1 - S0) / dt01;
    const double S_top = S0 - t0 * sig;
    double A[3], g0 = 0.0, g1 = 0.0;                    // surface terms of dL/dtau_0, dL/dtau_1
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double Gk = G * wmu[k];
        const ExpTerms64 et = exp_terms64(t0 / mu[k]);
        const double dCdx = S_top * et.e + (S0 - S_top) * et.dlw;
        const double dCdS = et.om - et.lw;
        g0 += Gk * (dCdx / mu[k] + dCdS * (-sig - t0 * sig / dt01));
        g1 += Gk * dCdS * (t0 * sig / dt01);
        A[k] = et.e;
    }
    // segments [j, j + 1]: ga to dL/dtau_j, gb to dL/dtau_{j+1}
    double Sa = S0, Sb = S1, ta = t0, tb = t1, chib = chi1, mb = m1;
    double pend = g1, last = 0.0;                      // pend: what depth j already holds
    for (int j = 0; j < D - 1; ++j) {
        if (j > 0) {
            const double mj = s.m[j + 1];
            const double chij = kc + col[(j + 1) * WAVE];
            Sa = Sb;
            ta = tb;
            Sb = p.planck(s.T[j + 1]);
            tb = ta + 0.5 * (chib + chij) * (mj - mb);
            chib = chij;
            mb = mj;
        }
        double ga = 0.0, gb = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const ExpTerms64 et = exp_terms64((tb - ta) / mu[k]);
            const double c = Sa * et.om + (Sb - Sa) * et.lw;
            const double dc = Sa * et.e + (Sb - Sa) * et.dlw;
            const double w = G * wmu[k] * A[k] / mu[k];
            ga -= w * (c + dc);
            gb += w * dc;
            A[k] *= et.e;
        }
        const double gj = (j == 0 ? g0 : pend) + ga;   // depth j is complete but for the bottom term
        if (j < D - 2)
            col[j * WAVE] = gj;
        else
            last = gj;
        pend = j == 0 ? g1 + gb : gb;
    }
    // bottom boundary (Sa, Sb, ta, tb are now the last segment)
    {
        const double dS = Sb - Sa, dtl = tb - ta;
        double g_last = 0.0, g_prev = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double Gk = G * wmu[k] * A[k];
            const double ID = Sb + mu[k] * dS / dtl;
            const double q = mu[k] * dS / (dtl * dtl);
            g_last += Gk * (-ID / mu[k] - q);
            g_prev += Gk * q;
        }
        col[(D - 2) * WAVE] = last + g_prev;
        col[(D - 1) * WAVE] = pend + g_last;
    }
    // dL/dchi_j from the trapezoid rule via suffix sums
    double suffix = 0.0, gnext = 0.0;
    float* out = s.gk + i;
    const size_t st = s.Npad;
    for (int j = D - 1; j >= 0; --j) {
        suffix += col[j * WAVE];
        double g = (j == D - 1) ? 0.0 : 0.5 * (s.m[j + 1] - s.m[j]) * gnext;
        g += (j == 0) ? s.m[0] * suffix : 0.5 * (s.m[j] - s.m[j - 1]) * suffix;
        out[(size_t)j * st] = (float)g;
        gnext = suffix;
    }
}

// A workgroup of WAVE pixels; col: the thread's column in LDS.
template <bool E2>
__device__ __forceinline__ void dev_flux_columns(const StarDev& s, int i, bool total, float* col) {
    if (total) {
        if (i < s.N) stage_kappa_column(s, i, col);
        E2 ? dev_flux_e2_column<true>(s, i, col) : dev_flux_column<true>(s, i, col);
    } else {
        E2 ? dev_flux_e2_column<false>(s, i, col) : dev_flux_column<false>(s, i, col);
    }
}

template <bool E2>
__device__ __forceinline__ void dev_reverse_columns(const StarDev& s, int i, double* col) {
    if (i < s.N) stage_kappa_column(s, i, col);
    E2 ? dev_reverse_e2_column(s, i, col) : dev_reverse_column(s, i, col);
}

// Whether a plan's transfer (reverse: its adjoint) goes by columns, by the times
// measured for both forms at 2-80 depths and 1,000-361,193 pixels (us; the
// models are within 15 % of them).  Rows cost their depth slots, 16 np a
// pixel; columns the serial walk of D depths, once for every 65,536 pixels or
// so that are in flight at a time.  72 depths, rows against columns:
//            Gauss-3 flux   adjoint     E2 flux     adjoint
//   10,000      21 / 52     42 / 116    27 / 61     22 / 66
//   80,000      77 / 94    211 / 234   134 / 119    99 / 125
//   361,193    321 / 317   953 / 739   596 / 447   431 / 378
// and 8 depths at 361,193: 82 / 49, 345 / 87, 241 / 60, 155 / 51.
inline bool columns_rule(int N, int D, int quad, bool reverse) {
    const double n = N, np = row_np(D), chunks = (D + 15) / 16, flights = std::ceil(n / 65536.0);
    if (quad == PZ_QUAD_E2)
        return reverse ? flights * (6.0 + 0.87 * D) < 7.0 + 2.35e-4 * n * np
                       : std::max(1.0, 0.6 + n / 50000.0) * (5.0 + 0.79 * D) < 7.0 + 3.35e-4 * n * np;
    return reverse ? flights * (7.0 + 1.55 * D) < 8.0 + 5.2e-4 * n * np
                   : flights * (5.9 + 0.65 * D) <
                         7.0 + 0.155 * D + std::max(0.0, n - 12000.0) * (9.5e-5 + 6.5e-5 * chunks + 6.2e-6 * D);
}

}  // namespace pz
