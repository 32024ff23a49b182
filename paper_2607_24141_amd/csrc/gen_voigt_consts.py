"""Writes voigt_consts.h: constants of the device Voigt evaluator.

Regions of z = v + i a (float32 unless noted):

* wing, |z| >= 5.5: Gauss-Hermite quadrature of the Voigt integral
  H(a,v) = (a/pi) int exp(-t^2)/((v-t)^2+a^2) dt with the +/-t_k node pairs
  combined so every term is positive,
      H ~= (2a/pi) sum_k w_k (u + a^2 + t_k^2) / ((u - a^2 - t_k^2)^2 + 4 u a^2),
  u = v^2.  Three tiers: 6 nodes for 5.5 <= |z| < 8, 4 nodes for
  8 <= |z| < 40, 2 nodes beyond (max relative error ~1.4e-6 in each).
* core with small damping, |z| < 5.5 and a <= 0.15: the expansion of
  w(v + ia) in powers of a about the real axis,
      w = exp(-z^2) + (2i/sqrt(pi)) F(z),   F = Dawson's integral,
      H = exp(a^2-u) cos(2av) - (2/sqrt(pi)) [a F' - a^3 F'''/6 + a^5 F^(5)/120]
      L = -exp(a^2-u) sin(2av) + (2/sqrt(pi)) [F - a^2 F''/2 + a^4 F''''/24].
  The Gaussian part carries the exact real-axis value, so H keeps its
  relative accuracy where exp(-v^2) and the damping term are comparable.
  The damping terms (derivatives of F, the even ones divided by v) are
  piecewise polynomials: |v| in [0, 5.5] is cut into PW_N intervals, and on
  each they are Chebyshev interpolants of degree 5, 4, 2 (for the a, a^3,
  a^5 terms) in t = |v| - (interval centre), from mpmath values at 40
  digits, stored as monomial coefficients (16 floats per interval, read from
  LDS): no division and short Horner chains.  For a <= A_TINY the a^5 terms
  are below 5e-8 of H and are dropped.
* core with larger damping: Weideman's 32-term rational expansion of w(z)
  (J.A.C. Weideman, SIAM J. Numer. Anal. 31 (1994) 1497) in float64.
* near zone of the split sums, a <= 0.15 and |v| < NEAR_V: with G(v) = 2 v F(v) - 1
  every damping term follows from g = (2/sqrt(pi)) G by recurrence (F' = -G,
  F^(n+1) = -2 v F^(n) - 2 n F^(n-1)):
      H = exp(a^2-u) cos(2av) + a [g + a^2 (s/3 + g (1 - 2u/3))
          + a^4 (s (7/30 - u/15) + g (1/2 - 2u/3 + 2u^2/15))],  s = 2/sqrt(pi),
  so one table serves H.  g is piecewise cubic in |v|
  (intervals of 1/NEAR_INV, Chebyshev nodes, 4 floats each).
* far zone of the split sums, v >= FAR_V and a <= FAR_AV v: with w = 1/v^2, b = a^2
      H = (a/sqrt(pi)) w sum_{n<=5} w^n P_n(b),
  P_n of degree n: the asymptotic coefficients of w(z) for n <= 3, the last two
  fitted (minimax on w <= 1/FAR_V^2, b w <= FAR_AV^2).  The same form with its
  own polynomials serves a dH/da, and X = H + a dH/da + v dH/dv with one
  more factor w (n <= 4 there).

Run:  python gen_voigt_consts.py > voigt_consts.h
"""
import numpy as np

N_W = 32
U_MAX = 30.25
A_SMALL = 0.15
A_TINY = 0.03      # a <= A_TINY: the a^5 terms (and the t^4 term of cos 2av) are dropped


def weideman(N):
    M = 2 * N
    k = np.arange(-M + 1, M)
    L = np.sqrt(N / np.sqrt(2.0))
    t = L * np.tan(k * np.pi / (2 * M))
    f = np.concatenate([[0.0], np.exp(-t * t) * (L * L + t * t)])
    a = np.real(np.fft.fft(np.fft.fftshift(f))) / (2 * M)
    return L, a[1:N + 1][::-1]          # highest power first (Horner order)


def dawson_derivs(v):
    """F, F', ..., F^(5) of Dawson's integral at v (mpmath, 40 digits)."""
    import mpmath as mp
    mp.mp.dps = 40
    out = np.zeros((6, len(v)))
    for i, x in enumerate(v):
        x = mp.mpf(x)
        F0 = mp.sqrt(mp.pi) / 2 * mp.exp(-x * x) * mp.erfi(x)
        d = [F0, 1 - 2 * x * F0]
        for n in range(1, 5):          # F^(n+1) = -2 v F^(n) - 2 n F^(n-1)
            d.append(-2 * x * d[n] - 2 * n * d[n - 1])
        out[:, i] = [float(y) for y in d]
    return out


PW_N = 16
PW_DEG = (5, 4, 2)


def pw_tables():
    """Per interval k of |v| in [0, U_MAX^(1/2)], for the damping terms of H (Lam) and
    of L/v (Mu): [P0_0..P0_3 | P0_4 P0_5 P2_0 P2_1 | P2_2 P2_3 P2_4 c | P4_0 P4_1 P4_2 0]
    with P0 ~ sum P0_n t^n (degree 5), P2 (degree 4), P4 (degree 2), t = |v| - c."""
    vmax = np.sqrt(U_MAX)
    h = vmax / PW_N
    sp = 2.0 / np.sqrt(np.pi)

    def terms(v):
        F = dawson_derivs(v)
        lam = [-sp * F[1], sp * F[3] / 6.0, -sp * F[5] / 120.0]
        mu = [sp * F[0] / v, -sp * F[2] / (2.0 * v), sp * F[4] / (24.0 * v)]
        return lam, mu

    tabs = np.zeros((2, PW_N, 16))
    for k in range(PW_N):
        c = (k + 0.5) * h
        for i, d in enumerate(PW_DEG):
            x = np.cos((2 * np.arange(d + 1) + 1) * np.pi / (2 * (d + 1)))
            t = 0.5 * h * x                      # Chebyshev nodes avoid v = 0 exactly
            lam, mu = terms(c + t)
            V = np.vander(t, d + 1, increasing=True)
            for j, y in enumerate((lam[i], mu[i])):
                co = np.linalg.solve(V, y)
                slot = (0, 6, 12)[i]
                tabs[j, k, slot:slot + d + 1] = co
        tabs[:, k, 11] = c
    # the layout above puts P2 at slots 6..10 and P4 at 12..14; c at 11
    return h, tabs[0], tabs[1]


def pw_check(h, tab):
    """Max relative error of the float32 piecewise H against wofz for a in (0, A_SMALL]."""
    from scipy.special import wofz
    f32 = np.float32
    t32 = tab.astype(f32)
    worst = {}
    for a, full in ((A_SMALL, True), (0.1, True), (A_TINY, False), (1e-2, False), (1e-3, False), (1e-5, False)):
        v = np.linspace(0.0, np.sqrt(U_MAX), 20001)[:-1]
        v = v[v * v + a * a < U_MAX]
        av = v.astype(f32)
        k = np.minimum((av * f32(1.0 / h)).astype(np.int32), PW_N - 1)
        T = t32[k]
        t = av - T[:, 11]
        L0 = T[:, 5]
        for n in (4, 3, 2, 1, 0):
            L0 = L0 * t + T[:, n]
        L2 = T[:, 10]
        for n in (9, 8, 7, 6):
            L2 = L2 * t + T[:, n]
        L4 = (T[:, 14] * t + T[:, 13]) * t + T[:, 12]
        a2 = f32(a * a)
        num = L0 + a2 * (L2 + a2 * L4) if full else L0 + a2 * L2
        u = av * av
        tt = f32(4) * a2 * u
        cs = 1 - tt / 2 + tt * tt / 24 - tt ** 3 / 720 + (tt ** 4 / 40320 if full else 0)
        H = np.exp(a2 - u).astype(np.float64) * cs + a * num.astype(np.float64)
        ref = wofz(v + 1j * a).real
        worst[a] = np.max(np.abs(H - ref) / ref)
    return worst


def pw_check_L(h, tab):
    """Max error of the float32 piecewise L = Im w relative to |w| (wofz)."""
    from scipy.special import wofz
    f32 = np.float32
    t32 = tab.astype(f32)
    worst = {}
    for a, full in ((A_SMALL, True), (0.1, True), (A_TINY, False), (1e-2, False), (1e-3, False)):
        v = np.linspace(0.0, np.sqrt(U_MAX), 20001)[:-1]
        v = v[v * v + a * a < U_MAX]
        av = v.astype(f32)
        k = np.minimum((av * f32(1.0 / h)).astype(np.int32), PW_N - 1)
        T = t32[k]
        t = av - T[:, 11]
        P0 = T[:, 5]
        for n in (4, 3, 2, 1, 0):
            P0 = P0 * t + T[:, n]
        P2 = T[:, 10]
        for n in (9, 8, 7, 6):
            P2 = P2 * t + T[:, n]
        P4 = (T[:, 14] * t + T[:, 13]) * t + T[:, 12]
        a2 = f32(a * a)
        num = P0 + a2 * (P2 + a2 * P4) if full else P0 + a2 * P2
        u = av * av
        tt = f32(4) * a2 * u
        sn = 1 - tt / 6 + tt * tt / 120 - tt ** 3 / 5040 + (tt ** 4 / 362880 if full else 0)
        L = v * (num.astype(np.float64) - np.exp(a2 - u).astype(np.float64) * 2 * a * sn)
        ref = wofz(v + 1j * a)
        worst[a] = np.max(np.abs(L - ref.imag) / np.abs(ref))
    return worst


NEAR_INV = 16
NEAR_V = 8.0
FAR_V = 5.5
FAR_AV = 0.2
FAR_N = 6          # powers w^1 .. w^6


def near_table():
    """Cubics of (2/sqrt(pi)) G in the fraction of each interval of |v|."""
    n = int(NEAR_V * NEAR_INV) + 1
    x = 0.5 * (1.0 - np.cos((np.arange(4) + 0.5) * np.pi / 4))
    tab = np.zeros((n, 4))
    for k in range(n):
        v = np.maximum((k + x) / NEAR_INV, 1e-30)
        tab[k] = np.linalg.solve(np.vander(x, 4, increasing=True), -2.0 / np.sqrt(np.pi) * dawson_derivs(v)[1])
    return tab


def near_check(tab):
    """Max relative error of the float32 near-zone H against wofz."""
    from scipy.special import wofz
    f = np.float32
    s = 2.0 / np.sqrt(np.pi)
    t32 = tab.astype(f)
    worst = {}
    for a in (A_SMALL, 0.1, A_TINY, 1e-2, 1e-3, 1e-5):
        v = np.linspace(0.0, NEAR_V, 40001)[:-1].astype(f)
        x = v * f(NEAR_INV)
        k = x.astype(np.int32)
        r = x - k.astype(f)
        q = t32[k]
        g = ((q[:, 3] * r + q[:, 2]) * r + q[:, 1]) * r + q[:, 0]
        u, a2 = v * v, f(a * a)
        h3 = f(s / 3) + g * (1 - f(2 / 3) * u)
        h5 = f(7 * s / 30) - f(s / 15) * u + g * (f(0.5) - f(2 / 3) * u + f(2 / 15) * u * u) if a > A_TINY else f(0)
        y = a2 * u
        cs = (((f(2 / 315) * y - f(4 / 45)) * y + f(2 / 3)) * y - 2) * y + 1
        H = np.exp2((a2 - u) * f(1.4426950408889634)).astype(np.float64) * cs + a * (g + a2 * (h3 + a2 * h5))
        ref = wofz(v.astype(np.float64) + 1j * np.sqrt(np.float64(a2))).real
        worst[a] = np.max(np.abs(H - ref) / ref)
    return worst


def far_fit(kind):
    """Polynomials of the far zone: coefficients {(m, k): c} of w^m (b w)^k and the max relative
    error.  kind 0: H, 1: a dH/da, 2: X / w."""
    from math import comb
    from scipy.special import wofz
    n, N = 60, FAR_N - 1
    ch = 0.5 * (1.0 - np.cos((np.arange(n) + 0.5) * np.pi / n))
    W, Q = (z.ravel() for z in np.meshgrid(ch / FAR_V ** 2, ch * FAR_AV ** 2, indexing="ij"))
    v = 1.0 / np.sqrt(W)
    a = np.sqrt(Q) * v
    z = wofz(v + 1j * a)
    H, L = z.real, z.imag
    aHa = 2.0 * a * (v * L + a * H) - 2.0 * a / np.sqrt(np.pi)
    X = H + aHa - 2.0 * v * (v * H - a * L)
    top = N if kind < 2 else N - 1
    y = (H, aHa, X / W)[kind] * np.sqrt(np.pi) / (a * W)
    exact = {}
    for m in range(N + 1):          # (2m-1)!!/2^m Re[i z^-(2m+1)], expanded in a/v
        dd = np.prod(np.arange(1.0, 2 * m, 2.0)) / 2.0 ** m
        for k in range(N + 1 - m):
            c = dd * comb(2 * m + 2 * k + 1, 2 * k + 1) * (-1.0) ** k
            if kind == 0:
                exact[m, k] = c
            elif kind == 1:
                exact[m, k] = c * (1 + 2 * k)
            elif m >= 1:
                exact[m - 1, k] = -2.0 * m * c
    keys = [(t - k, k) for t in range(top + 1) for k in range(t + 1)]
    out = {e: exact[e] for e in keys if sum(e) <= top - 2}
    free = [e for e in keys if e not in out]
    res = y - sum(c * W ** m * Q ** k for (m, k), c in out.items())
    A = np.stack([W ** m * Q ** k for m, k in free], 1) / y[:, None]
    sc = np.abs(A).max(0)
    wt = np.ones(y.size)
    for _ in range(60):
        c = np.linalg.lstsq(A / sc * wt[:, None], res / y * wt, rcond=None)[0]
        e = np.abs(A / sc @ c - res / y)
        wt = wt * (0.3 + e / e.max()) ** 0.3
        wt /= wt.mean()
    out.update(zip(free, c / sc))
    return out, e.max()


def far_arrays():
    out = []
    for kind, tag in ((0, "H"), (1, "A"), (2, "X")):
        c, err = far_fit(kind)
        top = max(m for m, _ in c)
        flat = [c[n - k, k] for n in range(top + 1) for k in range(n + 1)]
        out.append("/* far zone, %s: P_n, n = 0..%d, ascending powers of b; max relative error %.1e */"
                   % (("H", "a dH/da", "X")[kind], top, err))
        out.append(arr("PZ_FAR_%s" % tag, flat))
    return out


def arr(name, c, typ="float", fmt="%.9ef"):
    return "__device__ static constexpr %s %s[%d] = {%s};" % (typ, name, len(c), ", ".join(fmt % x for x in c))


def main():
    out = ["// Generated by gen_voigt_consts.py -- do not edit.", "#pragma once", ""]
    out.append("#define PZ_VOIGT_WING_R2 30.25f   /* |z|^2 below which the core formulas apply */")
    out.append("#define PZ_VOIGT_TIER2_R2 64.0f   /* |z| >= 8: four-node wing */")
    out.append("#define PZ_VOIGT_TIER3_R2 1600.0f /* |z| >= 40: two-node wing */")
    out.append("#define PZ_VOIGT_A2_SMALL %.6ef  /* a^2 <= this (a <= %.2f): float32 small-damping core */"
               % (A_SMALL ** 2, A_SMALL))
    out.append("#define PZ_VOIGT_A2_TINY %.6ef   /* a^2 <= this (a <= %.2f): core without the a^5 terms */"
               % (A_TINY ** 2, A_TINY))
    for n, tag in ((6, "GH6"), (4, "GH4"), (2, "GH2")):
        t, w = np.polynomial.hermite.hermgauss(n)
        pos = t > 0
        out.append(arr("PZ_%s_T2" % tag, t[pos] ** 2))
        out.append(arr("PZ_%s_W" % tag, w[pos] * 2.0 / np.pi) + "  /* w_k * 2/pi */")
    h, tab, tab_mu = pw_tables()
    worst = pw_check(h, tab)
    worst_l = pw_check_L(h, tab_mu)
    out.append("/* piecewise small-damping core, H terms: %d intervals of |v|, degrees %s; max relative error of H"
               % (PW_N, PW_DEG))
    out.append("   against wofz (float32 evaluation, includes the float32 exp): %s */"
               % ", ".join("a=%g: %.1e" % (k, v) for k, v in worst.items()))
    out.append("static constexpr int PZ_PW_N = %d;" % PW_N)
    out.append("#define PZ_PW_INV_H %.9ef" % (1.0 / h))
    out.append("__device__ static constexpr float PZ_PW_TAB[%d] = {" % (PW_N * 16))
    out += ["    " + ", ".join("%.9ef" % x for x in row) + "," for row in tab]
    out.append("};")
    out.append("/* the same for L = Im w (adjoint): max error of L relative to |w|: %s */"
               % ", ".join("a=%g: %.1e" % (k, v) for k, v in worst_l.items()))
    out.append("__device__ static constexpr float PZ_PW_MU_TAB[%d] = {" % (PW_N * 16))
    out += ["    " + ", ".join("%.9ef" % x for x in row) + "," for row in tab_mu]
    out.append("};")
    near = near_table()
    out.append("/* near zone: cubics of (2/sqrt(pi)) (2 v F(v) - 1), %d intervals of 1/%d; max relative error of H against"
               % (len(near), NEAR_INV))
    out.append("   wofz: %s */" % ", ".join("a=%g: %.1e" % (k, v) for k, v in near_check(near).items()))
    out.append("static constexpr int PZ_NEAR_N = %d;" % len(near))
    out.append("#define PZ_NEAR_INV %.1ff" % NEAR_INV)
    out.append("#define PZ_NEAR_V %.1ff" % NEAR_V)
    out.append("__device__ static constexpr float PZ_NEAR_TAB[%d] = {" % (4 * len(near)))
    out += ["    " + ", ".join("%.9ef" % x for x in row) + "," for row in near]
    out.append("};")
    out.append("#define PZ_FAR_V %.1f" % FAR_V)
    out.append("#define PZ_FAR_AV %.1f" % FAR_AV)
    out.append("static constexpr int PZ_FAR_N = %d;" % FAR_N)
    out += far_arrays()
    L, c = weideman(N_W)
    out.append("static constexpr int PZ_WEID_N = %d;" % N_W)
    out.append("#define PZ_WEID_L %.17e" % L)
    out.append("__device__ static constexpr double PZ_WEID_C[%d] = {" % N_W)
    out += ["    %.17e," % x for x in c]
    out.append("};")
    print("\n".join(out))


if __name__ == "__main__":
    main()
