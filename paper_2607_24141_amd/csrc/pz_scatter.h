// Transfer with continuum scattering (Sec. 2.1, Eqs. 3 and 6-8), per pixel in
// float64.  With sigma_c the scattering opacity per unit mass,
//   chi = kappa_abs + sigma_c,  eps = kappa_abs / chi,  S = eps B + (1 - eps) J,
// kappa_abs = kappa_c + sum kappa_line (total branch) or kappa_c (continuum
// branch).  J = Lambda S is the mean intensity of the discretised formal
// solution (piecewise-linear S in tau, linear extrapolation to tau = 0 over the
// surface segment, diffusion lower boundary I = S + mu dS/dtau; inward I = 0 at
// tau = 0), J_j = 1/2 sum_k w_k (I+_j(mu_k) + I-_j(mu_k)) on the 3-point
// Gauss-Legendre nodes of the flux.
//
// Forward: the fixed point S* = eps B + (1 - eps) Lambda S* by accelerated
// Lambda iteration (Jacobi with the diagonal Lambda*_jj of the same operator):
//   S <- S + (eps B + (1 - eps) Lambda S - S) / (1 - (1 - eps) Lambda*),
// from S = B until |dS_j| <= tol |S_j| at every depth (or the iteration cap),
// every fourth iteration followed by Ng's extrapolation from the last four
// iterates (Ng 1974: the combination of them whose next differences are
// smallest in the relative least-squares sense), then the emergent flux
// F = 2 pi sum_k w_k mu_k I+(0, mu_k).
//
// Backward (total branch): with gS = dF/dS* G and gtau the direct flux terms,
// the adjoint lambda solves (I - diag(1 - eps) Lambda)^T lambda = gS by the same
// preconditioned iteration with Lambda^T; then
//   dL/deps_j = lambda_j (B_j - J*_j),
//   dL/dtau  += VJP of J(S*, tau) with the cotangent (1 - eps) lambda,
//   dL/dchi   = trapezoid adjoint of dL/dtau,
//   dL/dkappa_line_j = dL/dchi_j + dL/deps_j sigma_j / chi_j^2.
//
// Layout: sixteen lanes (a row of the wavefront) per pixel, lane q holding the
// NP consecutive depths NP q .. NP q + NP - 1 and the segments that end at
// them, all three directions, in registers.  A sweep along depth is a linear
// recurrence I_j = e_j I_{j-1} + b_j: each lane runs its own NP steps, the rows
// combine by a four-step scan (row shifts; the multipliers are products of e,
// formed once per pixel), and each lane runs its steps again from its carry.
// The iteration so touches no memory: with one thread per (pixel, direction)
// and the segment coefficients in tables it moved 10.6 GB per launch at
// 37,550 pixels (2.0 ms; the adjoint 4.6 GB, 1.3 ms), bound by HBM.  What is
// left is float64 arithmetic, most of it the exponentials of the coefficients:
// at 20,011 pixels and 72 depths the forward takes 0.20 ms (1.18 before), the
// adjoint 0.11 (0.95).
// Segment j runs from depth j - 1 to j (j = 0: from the surface); with S between
// depths linear, e = e^-x, w = lw(x) and p = 1 - e^-x - lw(x):
//   inward   I_j     = e_j I_{j-1} + p_j S_j + w_j S_{j-1},
//   outward  I_{j-1} = e_j I_j + p_j S_{j-1} + w_j S_j.
#pragma once

namespace pz {

__device__ __forceinline__ double sc_mu(int k) { return k == 0 ? kMu0 : (k == 1 ? kMu1 : kMu2); }
__device__ __forceinline__ double sc_hw(int k) { return k == 1 ? 0.5 * 8.0 / 18.0 : 0.5 * 5.0 / 18.0; }   // w_k / 2

// One branch of one pixel, spread over its row.
template <int NP>
struct ScPixel {
    int D, q;                        // depths; lane of the row
    bool last;                       // holds depth D - 1
    int kd;                          // ... as its k = kd (uniform)
    double e[3][NP], p[3][NP], w[3][NP];   // segments; none past D - 1 (e = 1); lane 0: e_0 = 0, w_0 = 0, p_0 the weight of S_0 in I-_0
    double cw[3];                    // lane 0: -(the weight of S_1 in I-_0); else 0
    double P[3][4], Q[3][4];         // scan multipliers of the sweeps down and up
    double dt[NP];                   // tau_j - tau_{j-1} (j = 0: tau_0)
    double gd;                       // 1 / (tau_{D-1} - tau_{D-2}), in the last lane
    double eps[NP], inv[NP];         // eps and 1 / (1 - (1 - eps) Lambda*)
    double chi[NP];
    double kc, c1, c2, fs;

    __device__ __forceinline__ int depth(int k) const { return q * NP + k; }

    // S_{D-1} and S_{D-2} in the last lane (prev: the depth above the lane's first)
    __device__ __forceinline__ void bottom(const double* S, double prev, double& sd, double& sd2) const {
        sd = S[0];
        sd2 = prev;
#pragma unroll
        for (int k = 1; k < NP; ++k)
            if (k == kd) {
                sd = S[k];
                sd2 = S[k - 1];
            }
    }

    __device__ __forceinline__ double scan_down(int m, double r) const {
        r = fma(P[m][0], shr<1>(r), r);
        r = fma(P[m][1], shr<2>(r), r);
        r = fma(P[m][2], shr<4>(r), r);
        return fma(P[m][3], shr<8>(r), r);
    }
    __device__ __forceinline__ double scan_up(int m, double r) const {
        r = fma(Q[m][0], shl<1>(r), r);
        r = fma(Q[m][1], shl<2>(r), r);
        r = fma(Q[m][2], shl<4>(r), r);
        return fma(Q[m][3], shl<8>(r), r);
    }

    // I- of S along direction m at the lane's depths; prev = S above its first depth.
    __device__ __forceinline__ void inward(int m, const double* S, double prev, double* I) const {
        double b[NP], a = 0.0;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            b[k] = fma(S[k], p[m][k], (k ? S[k - 1] : prev) * w[m][k]);
            if (k == 0) b[0] = fma(-cw[m], S[1], b[0]);
            a = fma(e[m][k], a, b[k]);
        }
        double c = shr<1>(scan_down(m, a));
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            c = fma(e[m][k], c, b[k]);
            I[k] = c;
        }
    }

    // I+ of S along direction m at the lane's depths.
    __device__ __forceinline__ void outward(int m, const double* S, double prev, double* I) const {
        double sd, sd2;
        bottom(S, prev, sd, sd2);
        const double bnd = last ? fma(sc_mu(m) * gd, sd - sd2, sd) : 0.0;
        double b[NP], a = bnd;
#pragma unroll
        for (int k = NP - 1; k >= 0; --k) {
            b[k] = fma(k ? S[k - 1] : prev, p[m][k], S[k] * w[m][k]);
            a = fma(e[m][k], a, b[k]);
        }
        double c = shl<1>(scan_up(m, a));
        if (last) c = bnd;
#pragma unroll
        for (int k = NP - 1; k >= 0; --k) {
            I[k] = c;
            c = fma(e[m][k], c, b[k]);
        }
    }

    // J = Lambda S
    __device__ __forceinline__ void lambda(const double* S, double* J) const {
        const double prev = shr<1>(S[NP - 1]);
#pragma unroll
        for (int k = 0; k < NP; ++k) J[k] = 0.0;
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            double I[NP];
            inward(m, S, prev, I);
#pragma unroll
            for (int k = 0; k < NP; ++k) J[k] = fma(sc_hw(m), I[k], J[k]);
            outward(m, S, prev, I);
#pragma unroll
            for (int k = 0; k < NP; ++k) J[k] = fma(sc_hw(m), I[k], J[k]);
        }
    }

    // G_j = e_j G_{j-1} + v_j (down), at the lane's depths; in: G above its first depth
    __device__ __forceinline__ void adjoint_down(int m, const double* v, double* G, double& in) const {
        double a = 0.0;
#pragma unroll
        for (int k = 0; k < NP; ++k) a = fma(e[m][k], a, v[k]);
        double c = in = shr<1>(scan_down(m, a));
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            c = fma(e[m][k], c, v[k]);
            G[k] = c;
        }
    }
    // G_j = e_{j+1} G_{j+1} + v_j (up)
    __device__ __forceinline__ void adjoint_up(int m, const double* v, double* G) const {
        double a = 0.0;
#pragma unroll
        for (int k = NP - 1; k >= 0; --k) a = e[m][k] * (a + v[k]);
        double c = shl<1>(scan_up(m, a));
        if (last) c = 0.0;
#pragma unroll
        for (int k = NP - 1; k >= 0; --k) {
            G[k] = c + v[k];
            c = e[m][k] * G[k];
        }
    }

    // out += the transpose of S -> I+ along m for the down-swept G (gin above the lane): adds
    // G_{j-1} (p_j at j - 1, w_j at j) and the bottom boundary; what falls on the depth above the
    // lane's first goes to back.
    __device__ __forceinline__ void outward_T(int m, const double* G, double gin, double* out, double& back) const {
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const double g = k ? G[k - 1] : gin;
            out[k] = fma(g, w[m][k], out[k]);
            if (k)
                out[k - 1] = fma(g, p[m][k], out[k - 1]);
            else
                back = fma(g, p[m][0], back);
        }
        if (last) {
            const double f = sc_mu(m) * gd;
#pragma unroll
            for (int k = 0; k < NP; ++k)
                if (k == kd) {
                    out[k] = fma(G[k], 1.0 + f, out[k]);
                    if (k)
                        out[k - 1] = fma(-G[k], f, out[k - 1]);
                    else
                        back = fma(-G[k], f, back);
                }
        }
    }
    // out += the transpose of S -> I- along m for the up-swept G
    __device__ __forceinline__ void inward_T(int m, const double* G, double* out, double& back) const {
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            out[k] = fma(G[k], p[m][k], out[k]);
            if (k)
                out[k - 1] = fma(G[k], w[m][k], out[k - 1]);
            else
                back = fma(G[0], w[m][0], back);
        }
        out[1] = fma(-cw[m], G[0], out[1]);
    }

    // Lambda^T v
    __device__ __forceinline__ void lambda_T(const double* v, double* out) const {
        double back = 0.0;
#pragma unroll
        for (int k = 0; k < NP; ++k) out[k] = 0.0;
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            double h[NP], G[NP], in;
#pragma unroll
            for (int k = 0; k < NP; ++k) h[k] = sc_hw(m) * v[k];
            adjoint_down(m, h, G, in);
            outward_T(m, G, in, out, back);
            adjoint_up(m, h, G);
            inward_T(m, G, out, back);
        }
        out[NP - 1] += shl<1>(back);
    }

    // chi, eps, the segments and Lambda* of branch b at pixel i; B: Planck function at the lane's depths.
    __device__ __forceinline__ void setup(const StarDev& s, int i, int b, double* B) {
        D = s.D;
        q = threadIdx.x & 15;
        kd = (D - 1) % NP;
        last = q == (D - 1) / NP;
        const double lnl = log(s.lam_first_nm) + (double)i * s.h;
        const double lam_cm = exp(lnl) * 1.0e-7;
        kc = s.kappa0 * exp(s.alpha * (lnl - log(s.lam_ref_nm)));
        const double l2 = lam_cm * lam_cm;
        c1 = 2.0 * H_PLANCK * C_LIGHT * C_LIGHT / (l2 * l2 * lam_cm) * 1.0e-7;
        c2 = H_PLANCK * C_LIGHT / (lam_cm * K_BOLTZ);
        fs = exp(s.sigma_alpha * (lnl - log(s.lam_ref_nm)));
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int j = min(depth(k), D - 1);
            const double ka = kc + (b == 0 ? (double)s.kappa[(size_t)j * s.Npad + i] : 0.0);
            chi[k] = ka + s.sigma_c[j] * fs;
            eps[k] = ka / chi[k];
            B[k] = c1 / expm1(c2 / s.T[j]);
        }
        const double above = shr<1>(chi[NP - 1]);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int j = depth(k);
            const double mj = s.m[min(j, D - 1)];
            dt[k] = j == 0 ? chi[0] * mj : 0.5 * ((k ? chi[k - 1] : above) + chi[k]) * (mj - s.m[max(min(j, D - 1) - 1, 0)]);
        }
        {
            double d = dt[0];
#pragma unroll
            for (int k = 1; k < NP; ++k)
                if (k == kd) d = dt[k];
            gd = last ? 1.0 / d : 0.0;
        }
        const double c = q == 0 ? dt[0] / dt[1] : 0.0;    // tau_0 / (tau_1 - tau_0)
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const double imu = 1.0 / sc_mu(m);
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const ExpTerms64 t = exp_terms64(dt[k] * imu);
                const bool in = depth(k) < D;
                e[m][k] = in ? t.e : 1.0;
                p[m][k] = in ? t.om - t.lw : 0.0;
                w[m][k] = in ? t.lw : 0.0;
            }
            cw[m] = 0.0;
            if (q == 0) {                                 // the surface segment: S_top by extrapolation
                cw[m] = c * w[m][0];
                p[m][0] = p[m][0] + w[m][0] + cw[m];
                w[m][0] = 0.0;
                e[m][0] = 0.0;
            }
        }
        double L[NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) L[k] = 0.0;
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const double below = shl<1>(p[m][0]);         // the next lane's first segment
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                double out = k + 1 < NP ? p[m][k + 1] : below, in = p[m][k];
                if (last && k == kd) out = fma(sc_mu(m), gd, 1.0);
                // depth D - 2 and depth 1 share a boundary's extrapolation
                if (k == 1) in = fma(-e[m][1], cw[m], in);
                L[k] = fma(sc_hw(m), out + in, L[k]);
            }
            // Lambda*_{D-2} loses e_{D-1} mu / dtau of the diffusion boundary
            double x = 0.0;
            if (last)
#pragma unroll
                for (int k = 0; k < NP; ++k)
                    if (k == kd) {
                        const double f = sc_hw(m) * e[m][k] * sc_mu(m) * gd;
                        if (k)
                            L[k - 1] -= f;
                        else
                            x = f;
                    }
            L[NP - 1] -= shl<1>(x);
            double E = 1.0;
#pragma unroll
            for (int k = 0; k < NP; ++k) E *= e[m][k];
            double f = E, g = last ? 0.0 : E;
            P[m][0] = f;
            f *= shr<1>(f);
            P[m][1] = f;
            f *= shr<2>(f);
            P[m][2] = f;
            f *= shr<4>(f);
            P[m][3] = f;
            Q[m][0] = g;
            g *= shl<1>(g);
            Q[m][1] = g;
            g *= shl<2>(g);
            Q[m][2] = g;
            g *= shl<4>(g);
            Q[m][3] = g;
        }
#pragma unroll
        for (int k = 0; k < NP; ++k) inv[k] = 1.0 / (1.0 - (1.0 - eps[k]) * L[k]);
    }
};

// S* of the total branch, kept for the backward: [N][D].
__device__ __forceinline__ double* sc_source(const StarDev& s, int i) { return s.sc + (size_t)i * s.D; }

// Ng's extrapolation of S from x0 = S and the previous iterates x1, x2, x3:
// with d0 = x0 - x1, d1 = x1 - x2, d2 = x2 - x3 and weights 1/x0^2, (a, c)
// minimise |d0 - a (d0 - d1) - c (d0 - d2)|^2 and S <- (1 - a - c) x0 + a x1 +
// c x2; the one-term form (c = 0) when d0 - d1 and d0 - d2 are nearly parallel.
template <int NP>
__device__ __forceinline__ void sc_ng(const ScPixel<NP>& x, double* S, const double* x1, const double* x2,
                                      const double* x3, bool active) {
    double r[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < NP; ++k)
        if (x.depth(k) < x.D) {
            const double d0 = S[k] - x1[k], u = d0 - (x1[k] - x2[k]), v = d0 - (x2[k] - x3[k]);
            const double wt = 1.0 / (S[k] * S[k]);
            r[0] += wt * u * u;
            r[1] += wt * u * v;
            r[2] += wt * v * v;
            r[3] += wt * d0 * u;
            r[4] += wt * d0 * v;
        }
#pragma unroll
    for (int k = 0; k < 5; ++k) r[k] = row_sum(r[k]);
    const double det = r[0] * r[2] - r[1] * r[1];
    double a = 0.0, c = 0.0;
    if (det > 1e-10 * r[0] * r[2]) {
        a = (r[3] * r[2] - r[4] * r[1]) / det;
        c = (r[4] * r[0] - r[3] * r[1]) / det;
    } else if (r[0] > 0.0) {
        a = r[3] / r[0];
    }
    if (!(isfinite(a) && isfinite(c))) a = c = 0.0;
    if (active)
#pragma unroll
        for (int k = 0; k < NP; ++k) S[k] = (1.0 - a - c) * S[k] + a * x1[k] + c * x2[k];
}

// Forward of branch b at pixel i, one row of lanes (all 64 lanes of a
// wavefront call this; i beyond the grid computes the last pixel and stores
// nothing).  A pixel's S is frozen when it has converged, so its result does
// not depend on the wavefront's other pixels.
template <int NP>
__device__ __forceinline__ void dev_flux_scatter(const StarDev& s, int i, int b) {
    const bool px = i < s.N;
    i = min(i, s.N - 1);
    ScPixel<NP> x;
    double B[NP], S[NP], x1[NP], x2[NP], x3[NP];
    x.setup(s, i, b, B);
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        S[k] = x1[k] = x2[k] = x3[k] = B[k];
        B[k] *= x.eps[k];
    }
    bool active = true;
    int iters = 0;
    for (int it = 1;; ++it) {
        double J[NP];
        x.lambda(S, J);
        bool ok = true;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const double Sn = S[k] + (B[k] + (1.0 - x.eps[k]) * J[k] - S[k]) * x.inv[k];
            if (x.depth(k) < x.D && fabs(Sn - S[k]) > s.sc_tol * fabs(Sn)) ok = false;
            x3[k] = x2[k];
            x2[k] = x1[k];
            x1[k] = S[k];
            S[k] = active ? Sn : S[k];
        }
        if (active && (row_all(ok) || it >= s.sc_max_iter)) {
            active = false;
            iters = it;
        }
        if (!wave_any(active)) break;
        if (it % 4 == 0) sc_ng<NP>(x, S, x1, x2, x3, active);
    }
    const double prev = shr<1>(S[NP - 1]);
    double f = 0.0;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        double I[NP];
        x.outward(m, S, prev, I);
        if (x.q == 0) {                                   // through the surface segment
            const ExpTerms64 t = exp_terms64(x.dt[0] / sc_mu(m));
            const double S_top = S[0] - x.dt[0] * (S[1] - S[0]) / x.dt[1];
            f += 2.0 * PI * 2.0 * sc_hw(m) * sc_mu(m) * (I[0] * t.e + S_top * t.om + (S[0] - S_top) * t.lw);
        }
    }
    if (!px) return;
    if (x.q == 0) {
        float* out = b == 0 ? s.F : s.Fc;
        if (out) out[i] = (float)f;
        if (s.sc_iters) s.sc_iters[b * s.Npad + i] = iters;
    }
    if (b == 0)
#pragma unroll
        for (int k = 0; k < NP; ++k)
            if (x.depth(k) < x.D) sc_source(s, i)[x.depth(k)] = S[k];
}

// Backward of the total branch at pixel i, one row of lanes: needs the
// forward's S*; writes dL/dkappa_line into gk.  The adjoint iteration stops at
// max_j |d lambda_j| <= tol max_j |lambda_j| or the cap.
template <int NP>
__device__ __forceinline__ void dev_reverse_scatter(const StarDev& s, int i) {
    const bool px = i < s.N;
    i = min(i, s.N - 1);
    ScPixel<NP> x;
    double B[NP], S[NP];
    x.setup(s, i, 0, B);
#pragma unroll
    for (int k = 0; k < NP; ++k) S[k] = sc_source(s, i)[min(x.depth(k), x.D - 1)];
    const double Gseed = s.dLdF[i];
    const double prev = shr<1>(S[NP - 1]);
    // direct flux terms: dF/dS G into lam (the right-hand side), tau terms of the surface slab
    double rhs[NP], back = 0.0, top0 = 0.0, top1 = 0.0, src[3];
#pragma unroll
    for (int k = 0; k < NP; ++k) rhs[k] = 0.0;
    const double dt01 = x.dt[1], sig = (S[1] - S[0]) / dt01, t0 = x.dt[0], S_top = S[0] - t0 * sig;
    const double d0 = -sig - t0 * sig / dt01, d1 = t0 * sig / dt01;   // dS_top / dtau_0, dtau_1 (lane 0)
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const double mu = sc_mu(m), g0 = Gseed * 2.0 * PI * 2.0 * sc_hw(m) * mu;      // dL/dI(0, mu_m)
        src[m] = 0.0;
        if (x.q == 0) {
            const ExpTerms64 t = exp_terms64(t0 / mu);
            const double gStop = g0 * (t.om - t.lw);
            src[m] = g0 * t.e;                            // dL/dI+(tau_0)
            top0 += g0 * (S_top * t.e + (S[0] - S_top) * (t.e - t.lw * mu / t0)) / mu + gStop * d0;
            top1 += gStop * d1;
            rhs[0] += g0 * t.lw + gStop * (1.0 + t0 / dt01);
            rhs[1] += gStop * (-t0 / dt01);
        }
        double v[NP], G[NP], in;
#pragma unroll
        for (int k = 0; k < NP; ++k) v[k] = 0.0;
        v[0] = src[m];
        x.adjoint_down(m, v, G, in);
        x.outward_T(m, G, in, rhs, back);
    }
    rhs[NP - 1] += shl<1>(back);
    // adjoint fixed point: lambda = rhs + Lambda^T ((1 - eps) lambda)
    double lam[NP], U[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        if (x.depth(k) >= x.D) rhs[k] = 0.0;
        lam[k] = rhs[k];
        U[k] = (1.0 - x.eps[k]) * lam[k];
    }
    bool active = true;
    int iters = 0;
    for (int it = 1;; ++it) {
        double T[NP], dmax = 0.0, lmax = 0.0;
        x.lambda_T(U, T);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const double ln = x.depth(k) < x.D ? lam[k] + (rhs[k] + T[k] - lam[k]) * x.inv[k] : 0.0;
            dmax = fmax(dmax, fabs(ln - lam[k]));
            lmax = fmax(lmax, fabs(ln));
            if (active) {
                lam[k] = ln;
                U[k] = (1.0 - x.eps[k]) * ln;
            }
        }
        dmax = row_max(dmax);
        lmax = row_max(lmax);
        if (active && (dmax <= s.sc_tol * lmax || it >= s.sc_max_iter)) {
            active = false;
            iters = it;
        }
        if (!wave_any(active)) break;
    }
    // J* and the tau terms of the fixed point and of the flux
    double gt[NP], J[NP];
    back = 0.0;
#pragma unroll
    for (int k = 0; k < NP; ++k) gt[k] = J[k] = 0.0;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const double mu = sc_mu(m), hw = sc_hw(m), imu = 1.0 / mu;
        double Ip[NP], Im[NP], v[NP], G[NP], in;
        x.outward(m, S, prev, Ip);
        x.inward(m, S, prev, Im);
        const double Im_above = shr<1>(Im[NP - 1]);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            J[k] += hw * (Ip[k] + Im[k]);
            v[k] = hw * U[k];
        }
        if (x.q == 0) {
            top0 -= src[m] * Ip[0] * imu;
            v[0] += src[m];
        }
        // outward: G_{j-1} enters segment j
        x.adjoint_down(m, v, G, in);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            if (k == 0 && x.q == 0) continue;
            const double Sa = k ? S[k - 1] : prev, dlw = x.e[m][k] - x.w[m][k] * mu / x.dt[k];
            const double gx = x.depth(k) < x.D
                                  ? (k ? G[k - 1] : in) * (x.e[m][k] * (Sa - Ip[k]) + (S[k] - Sa) * dlw) * imu
                                  : 0.0;
            gt[k] += gx;
            if (k)
                gt[k - 1] -= gx;
            else
                back -= gx;
        }
        if (x.last) {
#pragma unroll
            for (int k = 0; k < NP; ++k)
                if (k == x.kd) {
                    const double dS = S[k] - (k ? S[k - 1] : prev);
                    const double g = G[k] * (-mu * dS * x.gd * x.gd);
                    gt[k] += g;
                    if (k)
                        gt[k - 1] -= g;
                    else
                        back -= g;
                }
        }
        // inward: G_j leaves segment j
#pragma unroll
        for (int k = 0; k < NP; ++k) v[k] = hw * U[k];
        x.adjoint_up(m, v, G);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            if (k == 0 && x.q == 0) {
                const ExpTerms64 t = exp_terms64(t0 * imu);
                top0 += G[0] * ((S[0] * t.e + (S_top - S[0]) * (t.e - t.lw * mu / t0)) * imu + t.lw * d0);
                top1 += G[0] * t.lw * d1;
                continue;
            }
            const double Sa = k ? S[k - 1] : prev, dlw = x.e[m][k] - x.w[m][k] * mu / x.dt[k];
            const double gx = x.depth(k) < x.D
                                  ? G[k] * (x.e[m][k] * (S[k] - (k ? Im[k - 1] : Im_above)) + (Sa - S[k]) * dlw) * imu
                                  : 0.0;
            gt[k] += gx;
            if (k)
                gt[k - 1] -= gx;
            else
                back -= gx;
        }
    }
    gt[NP - 1] += shl<1>(back);
    if (x.q == 0) {
        gt[0] += top0;
        gt[1] += top1;
    }
    if (x.q == 0 && px && s.sc_iters) s.sc_iters[2 * s.Npad + i] = iters;
    row_dchi<NP>(s, x.q, gt);
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const int j = x.depth(k);
        const double sg = s.sigma_c[min(j, x.D - 1)] * x.fs;
        const double geps = lam[k] * (B[k] - J[k]);
        if (px && j < x.D) s.gk[(size_t)j * s.Npad + i] = (float)(gt[k] + geps * sg / (x.chi[k] * x.chi[k]));
    }
}

}  // namespace pz
