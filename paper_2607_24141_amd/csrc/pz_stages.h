// Device bodies of every stage of the synthesis path.  The per-star kernels
// (pz_kernels.hip) and the persistent batch kernels (pz_batch.hip) call the
// same functions, so a batched star computes exactly what a per-star call
// computes.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "expint_consts.h"
#include "pz_internal.h"
#include "pz_rows.h"
#include "pz_voigt.h"

namespace pz {

static constexpr int WAVE = 64;

// ------------------------------------------------------------ populations
// Two-stage Saha ionisation (Sec. 3, Eq. 11) with no ionisation lowering:
//   Phi = (2 U_II / U_I) (2 pi m_e k T / h^2)^{3/2} exp(-chi / kT) / n_e,
//   f_I = 1/(1+Phi), f_II = Phi/(1+Phi); infinite chi => single stage.
// Output n_{s,r}/(rho U_{s,r}) with the abundance correction 10^dA (Eq. 30).
__device__ __forceinline__ void dev_populations(const StarDev& s, int idx) {
    if (idx == 0) s.wide_any[0] = 0;                  // raised by dev_line_consts
    if (idx >= s.S * s.D) return;
    const int sp = idx / s.D, j = idx - sp * s.D;
    const double T = s.T[j];
    const double chi = s.chi_ion[sp];
    const double U0 = s.U[(sp * 2 + 0) * s.D + j];
    const double U1 = s.U[(sp * 2 + 1) * s.D + j];
    const double saha = pow(2.0 * PI * M_ELECTRON * K_BOLTZ / (H_PLANCK * H_PLANCK), 1.5);
    double fI = 1.0, fII = 0.0;
    if (isfinite(chi)) {
        const double phi = 2.0 * U1 / U0 * saha * T * sqrt(T) * exp(-chi * EV_ERG / (K_BOLTZ * T)) / s.ne[j];
        if (phi <= 1.0) {
            fI = 1.0 / (1.0 + phi);
            fII = phi * fI;
        } else {
            fII = 1.0 / (1.0 + 1.0 / phi);
            fI = fII / phi;
        }
    }
    const double n = (s.dA ? exp10((double)s.dA[sp]) : 1.0) * s.n_species[sp * s.D + j];
    s.pop[(sp * 2 + 0) * s.D + j] = n * fI / (s.rho[j] * U0);
    s.pop[(sp * 2 + 1) * s.D + j] = n * fII / (s.rho[j] * U1);
    // reciprocal Doppler width (Eq. 5), per species and depth
    const double xi = (double)s.xi[0] * 1.0e5;
    s.inv_dv[sp * s.D + j] = 1.0 / sqrt(2.0 * K_BOLTZ * T / (s.mass[sp] * AMU_G) + xi * xi);
}

// ------------------------------------------------- line-selection keep test
// Per sorted line (Sec. 3, Eqs. 17-19), after dev_populations, in float64:
//   b     = floor(ln(lambda_l / lambda_first) / bin_ln) clamped to [0, B)
//   nu_b  = frequency at the bin's centre in ln lambda
//   C_jb  = eta kappa_c(nu_b) / (1 - exp(-h nu_b / k T_j))            (sigma_c = 0)
//   Q     = max_j pop_{s,r,j} / ((dv_{s,j} / c) C_jb)                  (pop = n / (rho U))
//   R_l   = sqrt(pi) e^2 / (m_e c) 10^(loggf + dgf) Q / nu_b
//   keep  = R_l >= 1 and R_l exp(-E_l / k T_deepest) >= 1
// Q is taken per line over the line's own (species, ion, bin): the same max
// over the same terms as a per-bin table, so no table is stored.
__device__ __forceinline__ void dev_select(const StarDev& s, int l, double eta, double bin_ln, int B,
                                           unsigned char* keep, double* R_out, double* Rd_out, int* n_keep) {
    if (l >= s.L) return;
    const int caller = s.ln.perm[l];
    const int spion = s.ln.spion[l], sp = spion >> 1;
    const double bf = floor(log(s.ln.lam_cm[l] * 1.0e7 / s.lam_first_nm) / bin_ln);
    const double b = fmin(fmax(bf, 0.0), (double)(B - 1));
    const double lam_b = s.lam_first_nm * exp((b + 0.5) * bin_ln);          // nm
    const double nu_b = C_LIGHT / (lam_b * 1.0e-7);
    const double kc = s.kappa0 * pow(lam_b / s.lam_ref_nm, s.alpha);
    double Q = 0.0;
    for (int j = 0; j < s.D; ++j) {
        const double C = eta * kc / (-expm1(-H_PLANCK * nu_b / (K_BOLTZ * s.T[j])));
        Q = fmax(Q, s.pop[spion * s.D + j] * s.inv_dv[sp * s.D + j] * C_LIGHT / C);
    }
    const double loggf = s.ln.loggf[l] + (s.dgf ? (double)s.dgf[caller] : 0.0);
    const double R = sqrt(PI) * E_CHARGE * E_CHARGE / (M_ELECTRON * C_LIGHT) * exp10(loggf) * Q / nu_b;
    const double Rd = R * exp(-s.ln.E_eV[l] * EV_ERG / (K_BOLTZ * s.T[s.D - 1]));
    const bool k = R >= 1.0 && Rd >= 1.0;
    if (keep) keep[caller] = k ? 1 : 0;
    if (R_out) R_out[caller] = R;
    if (Rd_out) Rd_out[caller] = Rd;
    if (k && n_keep) atomicAdd(n_keep, 1);
}

// ------------------------------------------------------ line-depth params
// Per line (Eqs. 4, 5, 30), in float64:
//   x = (pi e^2/m_e c) 10^(loggf+dgf) lambda_l / sqrt(pi)
//   y, z, w = 10^ddamp lambda_l / (4 pi) x (g_rad 10^d_rad, g_S 10^d_S, g_vdW 10^d_vdW)
// Block-wide maxima of n_e, n_pert and T over depth and of 1/dv over (species,
// depth).  They bound every line's damping width, damping ratio and Doppler
// width over depth.  Every thread of the workgroup calls this (it
// synchronises); red holds 4 doubles per thread.
struct DampBounds {
    double ne, npert, inv_dv, T;
};

__device__ __forceinline__ DampBounds damp_bounds(const StarDev& s, double* red) {
    const int t = threadIdx.x, n = blockDim.x;
    double a = 0.0, b = 0.0, c = 0.0, d = 0.0;
    for (int j = t; j < s.D; j += n) {
        a = fmax(a, s.ne[j]);
        b = fmax(b, s.npert[j]);
        d = fmax(d, s.T[j]);
    }
    for (int k = t; k < s.S * s.D; k += n) c = fmax(c, s.inv_dv[k]);
    red[t] = a;
    red[n + t] = b;
    red[2 * n + t] = c;
    red[3 * n + t] = d;
    __syncthreads();
    for (int w = n / 2; w > 0; w >>= 1) {
        if (t < w)
            for (int r = 0; r < 4; ++r) red[r * n + t] = fmax(red[r * n + t], red[r * n + t + w]);
        __syncthreads();
    }
    const DampBounds out = {red[0], red[n], red[2 * n], red[3 * n]};
    __syncthreads();
    return out;
}

// No pixel of a line's window has |x| above this: |lambda_l / lambda_i - 1| <=
// W / lambda_i <= W / (lambda_l - W), with room for rounding.
__device__ __forceinline__ float window_reach(const StarDev& s, double lam_cm) {
    const double den = lam_cm - s.window_cm;
    return den > 0.0 ? (float)(s.window_cm / den * (1.0 + 1.0e-4) + 1.0e-6) : INFINITY;
}

// bnd: damp_bounds of the workgroup.
__device__ __forceinline__ void dev_line_consts(const StarDev& s, int l, const DampBounds& bnd) {
    if (l >= s.L) return;
    const int caller = s.ln.perm[l];
    const double lam = s.ln.lam_cm[l];
    const double loggf = s.ln.loggf[l] + (s.dgf ? (double)s.dgf[caller] : 0.0);
    const double line_const = PI * E_CHARGE * E_CHARGE / (M_ELECTRON * C_LIGHT);
    const double damp = (s.ddamp ? exp10((double)s.ddamp[caller]) : 1.0) * lam / (4.0 * PI);
    const float* df = s.ddamp_family;                    // per-family corrections, [3][L] caller order
    const double4 c = make_double4(line_const * exp10(loggf) * lam / sqrt(PI),
                                   damp * exp10(s.ln.lgr[l] + (df ? (double)df[caller] : 0.0)),
                                   damp * exp10(s.ln.lgs[l] + (df ? (double)df[s.L + caller] : 0.0)),
                                   damp * exp10(s.ln.lgw[l] + (df ? (double)df[2 * s.L + caller] : 0.0)));
    s.lc[l] = c;
    const int sp = s.ln.spion[l] >> 1;
    const double gam = fma(c.w, bnd.npert, fma(c.z, bnd.ne, c.y));           // >= a dv at every depth
    // damping-ratio range over depth: flags lines whose wavefronts can mix near and far wing tiers
    bool wide = false, huge = false;
    if (gam * bnd.inv_dv > 1.0e3) {                        // else a <= 1000 at every depth
        double amin = 1e300, amax = 0.0;
        for (int j = 0; j < s.D; ++j) {
            const double a = fma(c.w, s.npert[j], fma(c.z, s.ne[j], c.y)) * s.inv_dv[sp * s.D + j];
            amin = fmin(amin, a);
            amax = fmax(amax, a);
        }
        wide = (amin < 8.0 && amax > 1.0e3) || (amin < 40.0 && amax > 3.0e4);
        huge = amax > 4.0e3;                               // a^10 of far_poly's polynomials: 3.5e37 there, past float32 at 5000
    }
    if (s.split) {
        // Far zone: v = x c / dv >= FAR_V at the widest dv, and a <= FAR_AV v,
        // i.e. x >= (a dv / c) / FAR_AV, at the largest damping width.
        const double xi = (double)s.xi[0] * 1.0e5;
        const double dv = sqrt(2.0 * K_BOLTZ * bnd.T / (s.mass[sp] * AMU_G) + xi * xi);
        float xfar = (float)(fmax(PZ_FAR_V * dv, gam / PZ_FAR_AV) / C_LIGHT * (1.0 + 1.0e-6));
        if (huge || !(xfar < window_reach(s, lam))) xfar = INFINITY;   // no far pixel in the window (or not a number)
        s.xfar[l] = wide ? -1.0f : xfar;
    } else {
        s.wide_a[l] = wide ? 1 : 0;
        if (wide) atomicOr(s.wide_any, 1);
    }
    if (s.center) {
        s.xlim[l] = 0.0f;                                // raised by dev_line_params
        s.inv_kcl[l] = 1.0 / (s.kappa0 * pow(lam * 1.0e7 / s.lam_ref_nm, s.alpha));   // 1 / kappa_c(lambda_l)
    }
}

// Per (line, depth), in float64 then rounded (Eqs. 4-5, 30):
//   dv = sqrt(2kT/m + xi^2),  dnu_D = dv / lambda_l
//   a  = 10^ddamp (g_rad + g_S n_e + g_vdW n_pert) / (4 pi dnu_D)
//   K  = (pi e^2/m_e c) n/(rho U) 10^(loggf+dgf) e^{-E/kT} (1 - e^{-h nu_l/kT}) / (sqrt(pi) dnu_D)
// stored as (c/dv, a^2, K, K a); v = (lambda_l/lambda_i - 1) c/dv.  The
// per-line and per-(species, depth) factors come from dev_line_consts and
// dev_populations.
// Every lane of the wavefront must call this (lanes past L*D included):
// the centre test reduces across the wavefront.
__device__ __forceinline__ void dev_line_params(const StarDev& s, long idx) {
    const long n = (long)s.L * s.D;                       // < 2^32 (the plan checks L D)
    const bool valid = idx < n;
    const unsigned id = (unsigned)(valid ? idx : n - 1);  // out-of-range lanes compute a copy, store nothing
    const int l = (int)(id / (unsigned)s.D), j = (int)(id - (unsigned)l * (unsigned)s.D);
    const double T = s.T[j];
    const int spion = s.ln.spion[l];
    const double inv_dv = s.inv_dv[(spion >> 1) * s.D + j];
    const double4 c = s.lc[l];
    const double a = fma(c.w, s.npert[j], fma(c.z, s.ne[j], c.y)) * inv_dv;
    const double ikT = 1.0 / (K_BOLTZ * T);
    const double K = c.x * s.pop[spion * s.D + j] * exp(-s.ln.E_eV[l] * EV_ERG * ikT) *
                     (-expm1(-(H_PLANCK * C_LIGHT) / s.ln.lam_cm[l] * ikT)) * inv_dv;
    const float4 q = make_float4((float)(C_LIGHT * inv_dv), (float)(a * a), (float)K, (float)(K * a));
    if (valid) s.lp[idx] = q;
    // a row that is not finite stays with the pixels of its own window: no far zone
    if (s.split && valid && !(fabsf(q.x) + q.y + fabsf(q.z) + fabsf(q.w) < INFINITY) && s.xfar[l] >= 0.0f) s.xfar[l] = INFINITY;
    if (!s.center) return;
    // continuum-referenced centre test, decided in float64: keep iff
    // K H(a,0) >= eta kappa_c(lambda_l); a kept pair deposits where
    // |v| <= V = max(sqrt(ln(R/eta)), sqrt(a R / (sqrt(pi) eta))), R = K / kappa_c
    const double eta = s.center_eta;
    const double R = K * s.inv_kcl[l];
    float zm = -1.0f, xl = 0.0f;
    if (R * __ocml_erfcx_f64(a) >= eta) {
        const double vd = R > eta ? sqrt(log(R / eta)) : 0.0;
        const double V = fmax(vd, sqrt(a * R / (sqrt(PI) * eta)));
        zm = (float)(V * V + a * a);
        xl = (float)(V / (C_LIGHT * inv_dv));              // detuning |x| = V dv / c
    }
    if (valid) s.zmax[idx] = zm;
    // a span that ends inside the window is cut pixel by pixel: no far zone
    if (s.split && valid && !(xl > window_reach(s, s.ln.lam_cm[l])) && s.xfar[l] >= 0.0f) s.xfar[l] = INFINITY;
    // Largest |x| over each line's depths: one wavefront-wide max and one
    // atomic per distinct line in the wavefront (non-negative floats order as
    // their bit patterns; the result does not depend on the order).
    const int lane = (int)(threadIdx.x & 63);
    bool done = !valid || !(xl > 0.0f);
    for (;;) {
        const unsigned long long b = __ballot(!done);
        if (b == 0) break;
        const int first = __ffsll(b) - 1;
        const int lc = __shfl(l, first, 64);
        float m = l == lc ? xl : 0.0f;
        for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
        if (lane == first) atomicMax(reinterpret_cast<int*>(&s.xlim[lc]), __float_as_int(m));
        if (l == lc) done = true;
    }
}

}  // namespace pz

#include "pz_opacity.h"
#include "pz_split.h"

namespace pz {

// ------------------------------------------------------- formal solution
// Piecewise-linear S(tau) between depths, diffusion lower boundary and a
// linear extrapolation of S to tau = 0 (Eq. 7), summed from the surface down:
//   I(0, mu) = C_top + sum_j A_j c_j + A_{D-1} I_D,
//   A_j = exp(-tau_j / mu),  x_j = (tau_{j+1} - tau_j)/mu,
//   c_j = S_j (1 - e^{-x_j}) + (S_{j+1} - S_j) lw(x_j),
//   lw(x) = (1 - (1 + x) e^{-x}) / x,
//   C_top = S_top (1 - e^{-x_t}) + (S_0 - S_top) lw(x_t), x_t = tau_0/mu,
//   S_top = S_0 - tau_0 (S_1 - S_0)/(tau_1 - tau_0),
//   I_D = S_{D-1} + mu (S_{D-1} - S_{D-2}) / (tau_{D-1} - tau_{D-2}).
// This is the bottom-up recurrence of the formal solution unrolled into a
// sum, so a single top-down pass with O(1) state per ray suffices.
// 3-point Gauss-Legendre on [0, 1]: mu = 1/2 -+ sqrt(3/5)/2, 1/2; w = 5/18, 8/18, 5/18
static constexpr double kMu0 = 0.1127016653792583, kMu1 = 0.5, kMu2 = 0.8872983346207417;
__constant__ float c_mu[3] = {(float)kMu0, (float)kMu1, (float)kMu2};
__constant__ float c_inv_mu[3] = {(float)(1.0 / kMu0), (float)(1.0 / kMu1), (float)(1.0 / kMu2)};
__constant__ float c_wmu[3] = {(float)(2.0 * PI * 5.0 / 18.0 * kMu0), (float)(2.0 * PI * 8.0 / 18.0 * kMu1),
                               (float)(2.0 * PI * 5.0 / 18.0 * kMu2)};  // 2 pi w_k mu_k

struct ExpTerms {
    float e, om, lw;        // e^-x, 1 - e^-x, lw(x)
};

__device__ __forceinline__ ExpTerms exp_terms(float x) {
    ExpTerms r;
    r.e = expf(-x);
    r.om = -expm1f(-x);
    if (x < 0.05f)          // series of lw (sum_{n>=2} (-1)^n (n-1) x^{n-1}/n!)
        r.lw = x * fmaf(x, fmaf(x, fmaf(x, fmaf(x, 1.0f / 144.0f, -1.0f / 30.0f), 0.125f), -1.0f / 3.0f), 0.5f);
    else
        r.lw = fmaf(-x, r.e, r.om) * (1.0f / x);
    return r;
}

struct PixelSetup {
    float kc;        // continuum per unit mass
    float c1;        // 2 h c^2 / lambda^5 per nm
    float c2;        // h c / (lambda k)
};

__device__ __forceinline__ PixelSetup pixel_setup(const StarDev& s, int i) {
    const double lnl = log(s.lam_first_nm) + (double)i * s.h;
    const double lam_cm = exp(lnl) * 1.0e-7;
    PixelSetup p;
    p.kc = (float)(s.kappa0 * exp(s.alpha * (lnl - log(s.lam_ref_nm))));
    const double l2 = lam_cm * lam_cm;
    p.c1 = (float)(2.0 * H_PLANCK * C_LIGHT * C_LIGHT / (l2 * l2 * lam_cm) * 1.0e-7);
    p.c2 = (float)(H_PLANCK * C_LIGHT / (lam_cm * K_BOLTZ));
    return p;
}

__device__ __forceinline__ float planck(const PixelSetup& p, float invT) {
    return p.c1 / expm1f(p.c2 * invT);
}

struct PixelSetup64 {
    double kc, c1, c2;                                    // as PixelSetup
    __device__ __forceinline__ double planck(double T) const { return c1 / expm1(c2 / T); }
};

__device__ __forceinline__ PixelSetup64 pixel_setup64(const StarDev& s, int i) {
    const double lnl = s.ln_first + (double)i * s.h;
    const double lam_cm = exp(lnl) * 1.0e-7, l2 = lam_cm * lam_cm;
    return {s.kappa0 * exp(s.alpha * (lnl - s.ln_ref)), 2.0 * H_PLANCK * C_LIGHT * C_LIGHT / (l2 * l2 * lam_cm) * 1.0e-7,
            H_PLANCK * C_LIGHT / (lam_cm * K_BOLTZ)};
}

// Both fluxes of the FLUX_PX pixels from i0 by a workgroup of 256, float32.
// What costs, the exponentials of a segment on three rays and two branches, is
// independent of the other segments and is spread over all lanes, sixteen
// depths at a time; only the running optical depth (one lane per pixel and
// branch) and F += A c, A *= e (one per pixel, branch and ray) walk the depths,
// over LDS and in depth order, so that the rounding is that of a scan by one
// thread: gradients of saturated spectra cancel to 1e-4 of their terms, and
// another order of these sums shows in them.  One thread per pixel and branch
// needs 72 serial steps with three rays' exponentials in each: 52 us at 1,795
// pixels, 16 now; 53 against 41 at 20,011.  Where one lane per pixel fills the
// chip the walk is no slower and dev_flux_column takes it (columns_rule).
constexpr int FLUX_PX = 16;
struct FluxLds {
    float kc[FLUX_PX], c1[FLUX_PX], c2[FLUX_PX];
    float invT[MAXD], m[MAXD];
    float S[MAXD][FLUX_PX];
    float tau[2][MAXD][FLUX_PX];                          // tau[0] holds chi first
    float2 t[2][3][16][FLUX_PX];                          // (c, e^-x) of sixteen segments
    float I[2][3][FLUX_PX];
};
__device__ __forceinline__ void dev_flux_block(const StarDev& s, int i0, FluxLds& L) {
    const int t = threadIdx.x, px = t & 15, g = t >> 4, D = s.D, i = min(i0 + px, s.N - 1);
    if (g == 0) {
        const PixelSetup p = pixel_setup(s, i);
        L.kc[px] = p.kc;
        L.c1[px] = p.c1;
        L.c2[px] = p.c2;
    }
    if (t >= 64 && t - 64 < D) {
        L.invT[t - 64] = (float)(1.0 / s.T[t - 64]);
        L.m[t - 64] = (float)s.m[t - 64];
    }
    __syncthreads();
    const PixelSetup p = {L.kc[px], L.c1[px], L.c2[px]};
    for (int j = g; j < D; j += 16) {
        L.S[j][px] = planck(p, L.invT[j]);
        L.tau[0][j][px] = p.kc + s.kappa[(size_t)j * s.Npad + i];
    }
    __syncthreads();
    if (g < 2) {
        float chi_b = g == 0 ? L.tau[0][0][px] : p.kc, tau = chi_b * L.m[0];
        L.tau[g][0][px] = tau;
#pragma unroll 8
        for (int j = 1; j < D; ++j) {
            const float chi = g == 0 ? L.tau[0][j][px] : p.kc;
            tau = fmaf(g == 0 ? 0.5f * (chi_b + chi) : p.kc, L.m[j] - L.m[j - 1], tau);
            L.tau[g][j][px] = tau;
            chi_b = chi;
        }
    }
    __syncthreads();
    // lanes of the walk: (branch, ray) = g < 6
    const int wb = g < 3 ? 0 : 1, wm = g - 3 * wb;
    float F = 0.0f, A = 1.0f;
    for (int j0 = 0; j0 < D; j0 += 16) {
        const int j = j0 + g;
        if (j < D) {
            const float Sb = L.S[j][px];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const float tb = L.tau[b][j][px];
                float Sa, dt;
                if (j == 0) {                             // the slab above the first depth
                    dt = tb;
                    Sa = Sb - tb * (L.S[1][px] - Sb) / (L.tau[b][1][px] - tb);
                } else {
                    dt = tb - L.tau[b][j - 1][px];
                    Sa = L.S[j - 1][px];
                }
#pragma unroll
                for (int m = 0; m < 3; ++m) {
                    const ExpTerms et = exp_terms(dt * c_inv_mu[m]);
                    L.t[b][m][g][px] = make_float2(fmaf(Sa, et.om, (Sb - Sa) * et.lw), et.e);
                }
            }
        }
        __syncthreads();
        if (g < 6) {
            const int n = min(16, D - j0);
            if (j0 == 0) F = L.t[wb][wm][0][px].x, A = L.t[wb][wm][0][px].y;
#pragma unroll 4
            for (int k = j0 == 0; k < n; ++k) {
                const float2 ce = L.t[wb][wm][k][px];
                F = fmaf(A, ce.x, F);
                A *= ce.y;
            }
        }
        __syncthreads();
    }
    if (g < 6) {
        const float Sa = L.S[D - 2][px], Sb = L.S[D - 1][px];
        const float grad = (Sb - Sa) / (L.tau[wb][D - 1][px] - L.tau[wb][D - 2][px]);
        L.I[wb][wm][px] = fmaf(A, fmaf(c_mu[wm], grad, Sb), F);
    }
    __syncthreads();
    if (g < 2 && i0 + px < s.N) {
        float out = 0.0f;
#pragma unroll
        for (int m = 0; m < 3; ++m) out = fmaf(c_wmu[m], L.I[g][m][px], out);
        (g == 0 ? s.F : s.Fc)[i] = out;
    }
    __syncthreads();                                      // L may be used again
}

// Float64 transfer quantities of a pixel on a row: opacity, segments, Planck function.
template <int NP>
struct RowPixel64 {
    int D, q, kd;
    bool last;
    double kc, S[NP], S_above;                            // S_above: S above the lane's first depth (lane 0: unset)
    double chi[NP], chi_above, dm[NP];

    __device__ __forceinline__ int depth(int k) const { return q * NP + k; }

    __device__ __forceinline__ void setup(const StarDev& s, int i) {
        D = s.D;
        q = threadIdx.x & 15;
        kd = (D - 1) % NP;
        last = q == (D - 1) / NP;
        const PixelSetup64 p = pixel_setup64(s, i);
        kc = p.kc;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int j = min(depth(k), D - 1);
            S[k] = p.planck(s.T[j]);
            chi[k] = kc + (double)s.kappa[(size_t)j * s.Npad + i];
            dm[k] = j == 0 ? s.m[0] : s.m[j] - s.m[j - 1];
        }
        S_above = shr<1>(S[NP - 1]);
        chi_above = shr<1>(chi[NP - 1]);
    }
    // tau_j - tau_{j-1} of the total (cont: the continuum) branch
    __device__ __forceinline__ void segments(bool cont, double* dt) const {
#pragma unroll
        for (int k = 0; k < NP; ++k)
            dt[k] = cont ? kc * dm[k]
                         : (depth(k) == 0 ? chi[0] : 0.5 * ((k ? chi[k - 1] : chi_above) + chi[k])) * dm[k];
    }
    // Value k = kd of an array (the last depth, in the last lane)
    __device__ __forceinline__ double at_kd(const double* a) const {
        double x = a[0];
#pragma unroll
        for (int k = 1; k < NP; ++k)
            if (k == kd) x = a[k];
        return x;
    }
};

// gt, dL/dtau at the lane's depths (0 past D - 1), becomes dL/dchi: the
// trapezoid rule's adjoint through the suffix sums Gamma_j.
template <int NP>
__device__ __forceinline__ void row_dchi(const StarDev& s, int q, double* gt) {
    const int D = s.D;
    double r = 0.0;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        if (q * NP + k >= D) gt[k] = 0.0;
        r += gt[k];
    }
    r += shl<1>(r);
    r += shl<2>(r);
    r += shl<4>(r);
    r += shl<8>(r);
    double next = shl<1>(r);                              // Gamma below the lane's last depth
#pragma unroll
    for (int k = NP - 1; k >= 0; --k) {
        const int j = min(q * NP + k, D - 1);
        const double suffix = next + gt[k];
        double g = j + 1 < D ? 0.5 * (s.m[j + 1] - s.m[j]) * next : 0.0;
        g += j == 0 ? s.m[0] * suffix : 0.5 * (s.m[j] - s.m[j - 1]) * suffix;
        gt[k] = g;
        next = suffix;
    }
}

template <int NP>
__device__ __forceinline__ void row_store_gk(const StarDev& s, int q, int i, const double* g) {
#pragma unroll
    for (int k = 0; k < NP; ++k)
        if (q * NP + k < s.D) s.gk[(size_t)(q * NP + k) * s.Npad + i] = (float)g[k];
}

// ------------------------------------------------------------ E2 quadrature
// E3(x) and E4(x) = (e^-x - x E3(x)) / 3 for x >= 0, float64 (the recurrence
// E_{n+1} = (e^-x - x E_n) / n; its cancellation for large x costs at most ~3
// of float64's 16 digits below x = 700, beyond which both are 0).  E3 is its
// power series up to x = 1 and e^-x / x times a polynomial in 1/x per octave
// beyond (expint_consts.h), to 7e-15 relative, as a series and a continued
// fraction summed to their ends are.  Those ends lie up to ninety divisions
// away near x = 1, and a wavefront waits for its slowest knot: 194 against 24 us
// for the flux, 85 against 17 for the adjoint (12,001 pixels, 72 depths).
__constant__ double c_e3_series[PZ_E3_SERIES_N] = {PZ_E3_SERIES};
__constant__ double c_e3_table[PZ_E3_OCTAVES * (PZ_E3_DEGREE + 1)] = {PZ_E3_TABLE};
__device__ __forceinline__ void expint34(double x, double& E3, double& E4) {
    if (x <= 0.0) {
        E3 = 0.5;
        E4 = 1.0 / 3.0;
        return;
    }
    if (x > 700.0) {
        E3 = 0.0;
        E4 = 0.0;
        return;
    }
    const double e = exp(-x);
    if (x <= 1.0) {
        double p = 0.0;
#pragma unroll
        for (int k = PZ_E3_SERIES_N - 1; k >= 0; --k) p = fma(p, x, c_e3_series[k]);
        E3 = 0.5 - x + x * x * fma(x, p, 0.5 * (PZ_E3_PSI - log(x)));
    } else {
        const double y = 1.0 / x;
        const int o = min(ilogb(x), PZ_E3_OCTAVES - 1);    // [2^o, 2^{o+1}); the last one open
        const double hi = ldexp(1.0, -o), lo = o == PZ_E3_OCTAVES - 1 ? 0.0 : 0.5 * hi;
        const double t = (y - lo) * (2.0 / (hi - lo)) - 1.0;
        const double* c = c_e3_table + max(o, 0) * (PZ_E3_DEGREE + 1);   // a NaN indexes row 0 and stays one
        double p = 0.0;
#pragma unroll
        for (int k = PZ_E3_DEGREE; k >= 0; --k) p = fma(p, t, c[k]);
        E3 = e * y * p;
    }
    E4 = (e - x * E3) * (1.0 / 3.0);
}

// E3 and E4 at the lane's knots tau_j, from its segments.
template <int NP>
__device__ __forceinline__ void row_expint(int D, int q, const double* dt, double* tau, double* E3, double* E4) {
    double r = 0.0;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        r += q * NP + k < D ? dt[k] : 0.0;
        tau[k] = r;
    }
    r += shr<1>(r);
    r += shr<2>(r);
    r += shr<4>(r);
    r += shr<8>(r);
    const double above = shr<1>(r);
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        tau[k] += above;
        E3[k] = E4[k] = 0.0;
        if (q * NP + k < D) expint34(tau[k], E3[k], E4[k]);
    }
}

// F = 2 pi int_0^inf S E2 dt for piecewise-linear S(tau): segment [ta, tb]
// with S = Sa + s (t - ta) adds Sa (E3(ta) - E3(tb)) + s (E4(ta) - E4(tb) - (tb - ta) E3(tb));
// below the last depth S continues linearly: S_D E3(tau_D) + s_D E4(tau_D);
// above the first depth the top slab runs from tau = 0 with the first slope.
// Both E2 fluxes of pixel i by a row of lanes, float64: every knot's
// exponential integrals and every segment are independent, so only the
// running optical depth and the final sum cross lanes.  12,001 pixels at 72
// depths: flux 453 us by one thread per pixel and the integrals' series, 194 by
// rows, 24 with the polynomials above; adjoint 450, 85 and 17.
template <int NP>
__device__ __forceinline__ void dev_flux_e2_row(const StarDev& s, int i) {
    const bool px = i < s.N;
    i = min(i, s.N - 1);
    RowPixel64<NP> x;
    x.setup(s, i);
#pragma unroll 1
    for (int b = 0; b < 2; ++b) {
        double dt[NP], tau[NP], E3[NP], E4[NP], F = 0.0;
        x.segments(b == 1, dt);
        row_expint<NP>(x.D, x.q, dt, tau, E3, E4);
        const double e3r = shr<1>(E3[NP - 1]), e4r = shr<1>(E4[NP - 1]);
        const double e3 = x.q ? e3r : 0.5, e4 = x.q ? e4r : 1.0 / 3.0;
        const double top = x.q ? x.S_above : x.S[0] - dt[0] * (x.S[1] - x.S[0]) / dt[1];
#pragma unroll
        for (int k = 0; k < NP; ++k)
            if (x.depth(k) < x.D) {
                const double Sa = k ? x.S[k - 1] : top, E3a = k ? E3[k - 1] : e3, E4a = k ? E4[k - 1] : e4;
                const double sl = (x.S[k] - Sa) / dt[k];
                F += Sa * (E3a - E3[k]) + sl * (E4a - E4[k] - dt[k] * E3[k]);
                if (x.last && k == x.kd) F += x.S[k] * E3[k] + sl * E4[k];      // S continues linearly below
            }
        F = 2.0 * PI * row_sum(F);
        if (x.q == 0 && px) (b == 0 ? s.F : s.Fc)[i] = (float)F;
    }
}

// Reverse of the E2 flux for the total branch.  With knots t_{-1} = 0,
// t_k = tau_k and slope s_k of segment k, the E2 terms of adjacent segments
// cancel at every knot (S is continuous), leaving
//   segment k >= 1:  dF/dtau_k     += -P_k s_k / dtau_k
//                    dF/dtau_{k-1} += s_k (E3(tau_k) - E3(tau_{k-1})) + P_k s_k / dtau_k,
//                    P_k = E4(t_{k-1}) - E4(t_k) - dtau_k E3(t_k);
//   top slab:        through E3(0) - E3(tau_0), P_0 and the extrapolated S_top;
//   bottom:          dF/dtau_{D-1} += -s_D E3 - E4 s_D/dtau, dF/dtau_{D-2} += E4 s_D/dtau;
// all times 2 pi; then the trapezoid suffix sums as for Gauss-3.
template <int NP>
__device__ __forceinline__ void dev_reverse_e2_row(const StarDev& s, int i) {
    const bool px = i < s.N;
    i = min(i, s.N - 1);
    RowPixel64<NP> x;
    x.setup(s, i);
    const double G = 2.0 * PI * (double)s.dLdF[i];
    double dt[NP], tau[NP], E3[NP], E4[NP], gt[NP], back = 0.0;
    x.segments(false, dt);
    row_expint<NP>(x.D, x.q, dt, tau, E3, E4);
    const double e3 = shr<1>(E3[NP - 1]), e4 = shr<1>(E4[NP - 1]);
#pragma unroll
    for (int k = 0; k < NP; ++k) gt[k] = 0.0;
    if (x.q == 0) {
        const double t0 = dt[0], d01 = dt[1], sig = (x.S[1] - x.S[0]) / d01;
        const double dE3 = 0.5 - E3[0];                   // E3(0) - E3(tau_0)
        const double P0 = 1.0 / 3.0 - E4[0] - t0 * E3[0]; // E4(0) - E4(tau_0) - tau_0 E3(tau_0)
        gt[0] = G * (dE3 * (-sig - t0 * sig / d01) + P0 * sig / d01);
        gt[1] = G * (dE3 * (t0 * sig / d01) - P0 * sig / d01);
    }
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const int j = x.depth(k);
        if (j == 0 || j >= x.D) continue;
        const double Sa = k ? x.S[k - 1] : x.S_above, E3a = k ? E3[k - 1] : e3, E4a = k ? E4[k - 1] : e4;
        const double sl = (x.S[k] - Sa) / dt[k];
        const double P = (E4a - E4[k] - dt[k] * E3[k]) * sl / dt[k];
        double up = G * (sl * (E3[k] - E3a) + P), down = -G * P;
        if (j == x.D - 1) {
            up += G * (E4[k] * sl / dt[k]);
            down += G * (-sl * E3[k] - E4[k] * sl / dt[k]);
        }
        gt[k] += down;
        if (k)
            gt[k - 1] += up;
        else
            back += up;
    }
    gt[NP - 1] += shl<1>(back);
    row_dchi<NP>(s, x.q, gt);
    if (px) row_store_gk<NP>(s, x.q, i, gt);
}

// ---------------------------------------------------------- reverse scan
// dL/dkappa_line[j][i] for the seed dL/dF_i (total branch only: the
// continuum branch depends on no correction).  dF/dtau_k is local in k in the
// summed form of the formal solution:
//   from A_k:           -A_k c_k / mu                        (k <= D-2)
//   from x_j:           +A_j c'_j / mu to tau_{j+1}, -A_j c'_j / mu to tau_j,
//                       c'_j = S_j e_j + (S_{j+1} - S_j) lw'(x_j)
//   bottom:             -A_{D-1} I_D / mu to tau_{D-1};  -/+ A_{D-1} mu dS/dtau^2
//   top slab:           via x_t and S_top (tau_0 and tau_1)
// then dL/dchi_j from the trapezoid tau scan by suffix sums Gamma_j.  The
// suffix sums are small differences of O(A S / mu) terms (S changes little
// between adjacent depths near the surface), so this scan runs in float64;
// only the result is rounded to float32.
struct ExpTerms64 {
    double e, om, lw, dlw;   // e^-x, 1 - e^-x, lw(x), lw'(x)
};

__device__ __forceinline__ ExpTerms64 exp_terms64(double x) {
    ExpTerms64 r;
    r.e = exp(-x);
    r.om = -expm1(-x);
    if (x < 1.0e-2) {
        // sum_{n>=2} (-1)^n (n-1) x^{n-1}/n! and its derivative, through n = 8
        double lw = 0.0, dlw = 0.0, fact = 2.0, xp = 1.0;
#pragma unroll
        for (int n = 2; n <= 8; ++n) {
            if (n > 2) fact *= n;
            const double sg = (n & 1) ? -1.0 : 1.0;
            dlw += sg * (n - 1) * (n - 1) * xp / fact;
            xp *= x;
            lw += sg * (n - 1) * xp / fact;
        }
        r.lw = lw;
        r.dlw = dlw;
    } else {
        r.lw = (r.om - x * r.e) / x;
        r.dlw = r.e - r.lw / x;
    }
    return r;
}

// By a row of lanes: a segment's transmission to the surface A_{j-1} is a
// product over all segments above, one scan per ray; the terms of the
// segments are then independent (72 depths, 1,795 pixels: 95 us by one thread
// per pixel, 16 now; 20,011 pixels: 98 against 61; from 120,000 pixels on, and
// at few depths, dev_reverse_column is the faster).
template <int NP>
__device__ __forceinline__ void dev_reverse_row(const StarDev& s, int i) {
    const bool px = i < s.N;
    i = min(i, s.N - 1);
    RowPixel64<NP> x;
    x.setup(s, i);
    const double G = s.dLdF[i];
    double dt[NP], gt[NP], back = 0.0;
    x.segments(false, dt);
#pragma unroll
    for (int k = 0; k < NP; ++k) gt[k] = 0.0;
    const double t0 = dt[0], dt01 = dt[1], sig = (x.S[1] - x.S[0]) / dt01, S_top = x.S[0] - t0 * sig;   // lane 0
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const double mu = m == 0 ? kMu0 : (m == 1 ? kMu1 : kMu2), imu = 1.0 / mu;
        const double Gw = G * 2.0 * PI * (m == 1 ? 8.0 / 18.0 : 5.0 / 18.0) * mu;
        ExpTerms64 t[NP];
        double r = 1.0;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            t[k] = exp_terms64(dt[k] * imu);
            r *= t[k].e;
        }
        // product of the lanes above
        double y = shr<1>(r);
        r = x.q >= 1 ? r * y : r;
        y = shr<2>(r);
        r = x.q >= 2 ? r * y : r;
        y = shr<4>(r);
        r = x.q >= 4 ? r * y : r;
        y = shr<8>(r);
        r = x.q >= 8 ? r * y : r;
        double A = shr<1>(r);
        if (x.q == 0) A = 1.0;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int j = x.depth(k);
            if (j == 0) {                                 // the surface slab
                const double dCdx = S_top * t[0].e + (x.S[0] - S_top) * t[0].dlw, dCdS = t[0].om - t[0].lw;
                gt[0] += Gw * (dCdx * imu + dCdS * (-sig - t0 * sig / dt01));
                gt[1] += Gw * dCdS * (t0 * sig / dt01);
            } else if (j < x.D) {
                const double Sa = k ? x.S[k - 1] : x.S_above, dS = x.S[k] - Sa;
                const double c = Sa * t[k].om + dS * t[k].lw, dc = Sa * t[k].e + dS * t[k].dlw;
                const double w = Gw * A * imu;
                double up = -w * (c + dc), down = w * dc;
                if (j == x.D - 1) {                       // the diffusion boundary
                    const double Gk = Gw * A * t[k].e, g = mu * dS / (dt[k] * dt[k]);
                    down += Gk * (-(x.S[k] + mu * dS / dt[k]) * imu - g);
                    up += Gk * g;
                }
                gt[k] += down;
                if (k)
                    gt[k - 1] += up;
                else
                    back += up;
            }
            A *= t[k].e;
        }
    }
    gt[NP - 1] += shl<1>(back);
    row_dchi<NP>(s, x.q, gt);
    if (px) row_store_gk<NP>(s, x.q, i, gt);
}

}  // namespace pz

#include "pz_columns.h"

namespace pz {

// Calls f with the depths per lane of D as a compile-time constant.
template <class F>
__host__ __device__ __forceinline__ void with_row_np(int D, F f) {
    switch (row_np(D)) {
        case 2: f(std::integral_constant<int, 2>()); break;
        case 3: f(std::integral_constant<int, 3>()); break;
        case 4: f(std::integral_constant<int, 4>()); break;
        default: f(std::integral_constant<int, 5>()); break;
    }
}

// -------------------------------------------------------- gather (adjoint)
// One wavefront per line: its lanes are 8 pixels x 8 depth groups and step
// through the window 8 pixels at a time; the line's per-depth parameters stay
// in registers.  The Voigt function and its derivatives are recomputed:
//   dL/d dgf   = ln10 sum g K H
//   dL/d ddamp = ln10 sum g K a dH/da
//   dL/d xi    = sum g (-K) (H + a dH/da + v dH/dv) d ln dnu_D / d xi,
//   d ln dnu_D / d xi = xi / dv^2 = xi (s / c)^2 with s = c/dv  (per km/s: x 1e10)
// A fixed-order butterfly reduces across lanes, so the sums are deterministic.
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, WAVE);
    return x;
}

// Far-wing series for the gather, |z|^2 = v^2 + a^2 >= 64 and b = a^2 <= 4.
// The asymptotic expansion w(z) ~ (i/sqrt(pi)) sum_n (2n-1)!!/2^n z^-(2n+1),
// its real part re-expanded in r = 1/|z|^2 (Im z^(2n+1) = a sum_j
// C(2n+1, 2j+1) (-b)^j (1/r - b)^(n-j)), gives with d|z|^2/da = 2a and
// d|z|^2/dv = 2v
//   H       = (a/sqrt(pi)) r sum_m e_m r^m,
//   a dH/da = (a/sqrt(pi)) r sum_m (e_m + 2b e_m' - 2b m e_(m-1)) r^m,
//   X = H + a dH/da + v dH/dv = (a/sqrt(pi)) r sum_(m>=1) (2b e_m' - 2m e_m) r^m,
// e_0 = 1, e_1 = 3/2, e_2 = 15/4 - 2b, e_3 = 105/8 - 15b,
// e_4 = 945/16 - 105b + 12b^2 (X's leading orders cancel in closed form).
// Cut after r^4, in float32, against the float64 Faddeeva function over
// |z| >= 8, b <= 4: H within 6.9e-7, a dH/da 1.5e-5, X 9.1e-5 relative (the
// node-pair sums: 1e-6, 1e-6, 1.6e-4), in 34 operations against 43.
static constexpr float kFarZ2 = 64.0f, kFarB = 4.0f;

// The series' sums: H = c r ph, a dH/da = c r pa, X = c r^2 px, c = a/sqrt(pi).
__device__ __forceinline__ void far_series(float b, float z2, float& r, float& ph, float& pa, float& px) {
    r = __builtin_amdgcn_rcpf(z2);
    const float e2 = fmaf(-2.0f, b, 3.75f), e3 = fmaf(-15.0f, b, 13.125f);
    const float e4 = fmaf(fmaf(12.0f, b, -105.0f), b, 59.0625f);
    const float f1 = fmaf(-2.0f, b, 1.5f), f2 = fmaf(-12.0f, b, 3.75f);
    const float f3 = fmaf(fmaf(12.0f, b, -67.5f), b, 13.125f);
    const float f4 = fmaf(fmaf(180.0f, b, -420.0f), b, 59.0625f);
    const float g2 = fmaf(4.0f, b, -15.0f), g3 = fmaf(60.0f, b, -78.75f);
    const float g4 = fmaf(fmaf(-48.0f, b, 630.0f), b, -472.5f);
    ph = fmaf(fmaf(fmaf(fmaf(e4, r, e3), r, e2), r, 1.5f), r, 1.0f);
    pa = fmaf(fmaf(fmaf(fmaf(f4, r, f3), r, f2), r, f1), r, 1.0f);
    px = fmaf(fmaf(fmaf(g4, r, g3), r, g2), r, -3.0f);
}

// One call per wavefront; l must be wavefront-uniform; pw holds the H and L
// core tables and lq the line's rows written by stage_line_params (both LDS).
// A step whose lanes are all at |z|^2 >= 64 with a^2 <= 4 takes the far-wing
// series, other steps voigt_KHD.
// FAM: the damping term is split over the three families by their share of
// the width at each depth, w_beta = Gamma_beta / Gamma.
// NEAR: the near zone only; the far zone's sums are in gline (dev_gather_far).
template <bool CT, bool FAM, bool NEAR>
__device__ __forceinline__ void gather_body(const StarDev& s, int l, int lane, const float4* pw, const float4* lq) {
    constexpr int WPX = 8, NDG = 8, DPT = (MAXD + NDG - 1) / NDG;
    const int px = lane % WPX, dg = lane / WPX;
    int ilo = s.ln.ilo[l], ihi = s.ln.ihi[l];
    const int ic = s.ln.ic[l];
    const float delta = s.ln.delta[l];
    const int D = s.D;
    const float4* lp = lq;
    const float* zm = CT ? s.zmax + (size_t)l * D : nullptr;
    if (CT) {
        // pixels whose detuning x = expm1(delta - k h) can reach the line's
        // largest span: |x| <= xl  <=>  delta - k h in [log1p(-xl), log1p(xl)]
        const double xl = (double)s.xlim[l] * (1.0 + 1e-5);
        if (!(xl > 0.0)) {
            ihi = ilo - 1;                                // no depth kept
        } else if (xl < 1e-2) {
            const double h = s.h, dl = (double)delta;
            ilo = max(ilo, ic + (int)floor((dl - log1p(xl)) / h) - 1);
            ihi = min(ihi, ic + (int)ceil((dl - log1p(-xl)) / h) + 1);
        }
    }
    const float reach = NEAR ? near_reach(s.xfar[l]) : INFINITY;
    if (NEAR) {
        // pixels with |x| < reach lie within (reach + reach^2) / h + 1/2 of the anchor
        const float w = fmaf(reach, reach, reach) / s.h_hi + 2.0f;
        if (reach < 0.5f && w < 1.0e6f) {
            ilo = max(ilo, ic - (int)w);
            ihi = min(ihi, ic + (int)w);
        }
    }
    float sgf = 0.0f, sd = 0.0f, sxi = 0.0f, sds = 0.0f, sdw = 0.0f;
    for (int p0 = ilo; p0 <= ihi; p0 += WPX) {
        const int i = p0 + px;
        const float x = detuning(i - ic, delta, s.h_hi, s.h_lo);
        if (i <= ihi && (!NEAR || fabsf(x) < reach)) {
            const float* g = s.gk + i;
#pragma unroll 1
            for (int d = 0; d < DPT; ++d) {
                const int j = d * NDG + dg;
                if (j < D) {
                    const float4 q = lp[j];
                    const float v = x * q.x;
                    if (CT && !(fmaf(v, v, q.y) <= zm[j])) continue;
                    const float gj = g[(size_t)j * s.Npad];
                    const float u = v * v, z2 = u + q.y;
                    const float4 e = lp[MAXD + j];
                    // g K H = w th, g K a dH/da = w ta, g K X e.x = w tx
                    float w, th, ta, tx;
                    if (wave_all(z2 >= kFarZ2) && wave_all(q.y <= kFarB)) {
                        float r;
                        far_series(q.y, z2, r, th, ta, tx);
                        w = (gj * r) * (q.w * kInvSqrtPiF);
                        tx *= r * e.x;
                    } else {
                        voigt_KHD(q.y, q.z, q.w, v, u, pw, th, ta, tx);
                        w = gj;
                        tx *= e.x;
                    }
                    sgf = fmaf(w, th, sgf);
                    sxi = fmaf(w, tx, sxi);
                    if (FAM) {
                        const float t = w * ta;
                        sd = fmaf(t, e.y, sd);
                        sds = fmaf(t, e.z, sds);
                        sdw = fmaf(t, e.w, sdw);
                    } else {
                        sd = fmaf(w, ta, sd);
                    }
                }
            }
        }
    }
    sgf = wave_sum(sgf);
    sd = wave_sum(sd);
    sxi = wave_sum(sxi);
    if (FAM) {
        sds = wave_sum(sds);
        sdw = wave_sum(sdw);
    }
    if (lane == 0) {
        if (NEAR) {
            sgf += s.gline[l];
            sd += s.gline[s.L + l];
            sxi += s.gline[2 * s.L + l];
            if (FAM) {
                sds += s.gline[3 * s.L + l];
                sdw += s.gline[4 * s.L + l];
            }
        }
        s.gline[l] = (float)LN10 * sgf;
        s.gline[s.L + l] = (float)LN10 * sd;
        s.gline[2 * s.L + l] = sxi;
        if (FAM) {
            s.gline[3 * s.L + l] = (float)LN10 * sds;
            s.gline[4 * s.L + l] = (float)LN10 * sdw;
        }
    }
}

template <bool NEAR>
__device__ __forceinline__ void dev_gather(const StarDev& s, int l, int lane, const float4* pw, const float4* lq) {
    if (l >= s.L) return;
    if (s.fam) {
        if (s.center)
            gather_body<true, true, NEAR>(s, l, lane, pw, lq);
        else
            gather_body<false, true, NEAR>(s, l, lane, pw, lq);
    } else {
        if (s.center)
            gather_body<true, false, NEAR>(s, l, lane, pw, lq);
        else
            gather_body<false, false, NEAR>(s, l, lane, pw, lq);
    }
}

// A wavefront copies line l's per-depth parameters to its LDS rows (l must
// be wavefront-uniform; nothing for l >= L): lq[j] = (c/dv, a^2, K, K a) and
// lq[MAXD + j] = (-xi (c/dv)^2 per km/s -- the microturbulence factor of the
// xi term, with its sign -- and, with damping families, the radiative, Stark
// and van der Waals shares of the width at depth j).
__device__ __forceinline__ void stage_line_params(const StarDev& s, int l, int lane, float4* lq) {
    if (l >= s.L) return;
    const float xi_f = s.xi[0] * (float)(1.0e10 / (C_LIGHT * C_LIGHT));
    float gr = 0.0f, gs = 0.0f, gw = 0.0f;
    if (s.fam) {
        const double4 c = s.lc[l];
        gr = (float)c.y;
        gs = (float)c.z;
        gw = (float)c.w;
    }
    for (int k = lane; k < s.D; k += WAVE) {
        const float4 q = s.lp[(size_t)l * s.D + k];
        lq[k] = q;
        float4 e = make_float4(-xi_f * q.x * q.x, 0.0f, 0.0f, 0.0f);
        if (s.fam) {
            const float Gs = gs * (float)s.ne[k], Gw = gw * (float)s.npert[k];
            const float inv = 1.0f / (gr + Gs + Gw);
            e.y = gr * inv;
            e.z = Gs * inv;
            e.w = Gw * inv;
        }
        lq[MAXD + k] = e;
    }
}

}  // namespace pz

#include "pz_split_gather.h"

namespace pz {

// ----------------------------------------------------------- reductions
__device__ __forceinline__ void dev_scatter(const StarDev& s, int l) {
    if (l >= s.L) return;
    const int c = s.ln.perm[l];
    if (s.g_loggf) s.g_loggf[c] = s.gline[l];
    if (s.g_damp) {
        s.g_damp[c] = s.gline[s.L + l];
        if (s.fam) {                                      // [3][L]: radiative, Stark, van der Waals
            s.g_damp[s.L + c] = s.gline[3 * s.L + l];
            s.g_damp[2 * s.L + c] = s.gline[4 * s.L + l];
        }
    }
}

// Abundance gradient of species b = sum of the dgf gradients of its lines
// (10^dA and 10^dgf scale the same strength at fixed atmosphere);
// microturbulence = sum of the per-line terms.  Two fixed-order levels:
// block (c, b) sums chunk c (RCHUNK lines) of list b into partial[b][c]
// (b = S is the xi list), then one block per list sums its partials.
__device__ __forceinline__ float block_sum256(float acc, float* red) {
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    return red[0];
}

// 256-thread workgroups.
__device__ __forceinline__ void dev_reduce_partial(const StarDev& s, int c, int b, float* red) {
    int o0, o1;
    if (b < s.S) {
        o0 = s.sp_off[b] + c * RCHUNK;
        o1 = min(s.sp_off[b + 1], o0 + RCHUNK);
    } else {
        o0 = c * RCHUNK;
        o1 = min(s.L, o0 + RCHUNK);
    }
    if (o0 >= o1) {
        if (threadIdx.x == 0) s.partial[b * s.n_rchunk + c] = 0.0f;
        return;
    }
    float acc = 0.0f;
    if (b < s.S) {
        for (int k = o0 + threadIdx.x; k < o1; k += 256) acc += s.gline[s.sp_idx[k]];
    } else {
        for (int k = o0 + threadIdx.x; k < o1; k += 256) acc += s.gline[2 * s.L + k];
    }
    const float tot = block_sum256(acc, red);
    if (threadIdx.x == 0) s.partial[b * s.n_rchunk + c] = tot;
}

__device__ __forceinline__ void dev_reduce_final(const StarDev& s, int b, float* red) {
    float acc = 0.0f;
    for (int c = threadIdx.x; c < s.n_rchunk; c += 256) acc += s.partial[b * s.n_rchunk + c];
    const float tot = block_sum256(acc, red);
    if (threadIdx.x == 0) {
        if (b < s.S) {
            if (s.g_abund) s.g_abund[b] = tot;
        } else if (s.g_xi) {
            s.g_xi[0] = tot;
        }
    }
}

// ------------------------------------------------------------- loss seed
// f = F/Fc, r = 2 (f - y)/sigma^2: dL/dF = r/Fc, dL/dFc = -r F/Fc^2.
__device__ __forceinline__ void dev_chi2_seed(int N, const float* F, const float* Fc, const float* y, float inv_s2,
                                              float* gF, float* gFc, int i) {
    if (i >= N) return;
    const float inv_c = 1.0f / Fc[i];
    const float f = F[i] * inv_c;
    const float r = 2.0f * (f - y[i]) * inv_s2;
    gF[i] = r * inv_c;
    if (gFc) gFc[i] = -r * f * inv_c;
}

// One 1024-thread workgroup: fixed-order sum of ((f - y)/sigma)^2.
__device__ __forceinline__ void dev_chi2_loss(int N, const float* F, const float* Fc, const float* y, float inv_s2,
                                              float* loss, float* red) {
    float acc = 0.0f;
    for (int i = threadIdx.x; i < N; i += 1024) {
        const float d = F[i] / Fc[i] - y[i];
        acc = fmaf(d * d, inv_s2, acc);
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = red[0];
}

}  // namespace pz
