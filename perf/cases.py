"""Timed work of the synthesis library: whole calls through its public entry points.

A case is one call, or one fitting step, that a program makes over and over: a
forward spectrum, a spectrum with the gradients of a fit, a batch of stars, the
instrument operator, one evaluation of the line calibration.  Sizes are those
of the library's workloads (500-503 nm with 1,000 lines; 1500-1700 nm with
200,000 lines; 300-1000 nm with 5,000,000; stars of 5,000-37,550 pixels and
10,000-200,000 lines; APOGEE-like observed pixels; 42,886 catalogue records)
and generic ones between them, odd ones among them.

exact() computes the same outputs in float64 with plain torch.
"""
import math
from types import SimpleNamespace as NS

import numpy as np
import torch

import paper_2607_24141_amd as pz

C = 2.99792458e10
C_KMS = 299792.458
H = 6.62607015e-27
KB = 1.380649e-16
QE = 4.803204712570263e-10
ME = 9.1093837015e-28
AMU = 1.66053906660e-24
EV = 1.602176634e-12
LN10 = math.log(10.0)
W_NM = 0.3
R_GRID = 3.0e5
SIGMA = 0.01                        # noise level of the chi^2 fits

# ------------------------------------------------------------------- the cases
SYNTH = dict(kind="synth", lam=1500.0, N=37550, L=200000, S=20, D=72, teff=4500.0, logg=2.5, xi=1.7, bands=0.3,
             step="fwd", quad="gauss3", eta=0.0, fam=False, sigma_c=0.0, tile=0)


def _synth(name, **kw):
    return dict(SYNTH, name=name, **kw)


def listed():
    return [
        # the smallest call: a narrow solar interval, one spectrum (launch latency, a few tiles)
        _synth("fwd_500nm", lam=500.0, N=1795, L=1000, S=10, teff=5777.0, logg=4.44, xi=0.7, bands=0.0),
        # the same size inside a torch program: gradients of a chi^2 through torch.autograd
        _synth("autograd_500nm", lam=517.0, N=1361, L=777, S=10, D=64, teff=5777.0, logg=4.44, xi=1.1, bands=0.0,
               step="autograd"),
        # the survey interval, one spectrum, with the tile width that the autotuner picks there
        _synth("fwd_hband", tile=32),
        # the same interval, one step of a fit of all corrections: spectrum, chi^2 seed, gradients
        _synth("fit_hband", step="fit"),
        # the widest interval: 361,193 pixels and five million lines, one spectrum
        _synth("fwd_optical", lam=300.0, N=361193, L=5000000, S=40, teff=5777.0, logg=4.44, xi=0.7, bands=0.0, tile=32),
        # a blue interval with wide windows in pixels, one fitting step, ragged sizes
        _synth("fit_blue", lam=427.0, N=18743, L=60013, S=30, teff=6100.0, logg=4.2, xi=1.3, bands=0.0, step="fit"),
        # the exact angle integral (E2, float64 transfer), one fitting step on part of the survey interval
        _synth("fit_e2", lam=1530.0, N=12001, L=40000, step="fit", quad="e2"),
        # continuum scattering (source function iterated in float64), one fitting step
        _synth("fit_scatter", N=20011, L=80000, step="fit", sigma_c=0.5),
        # the centre test with gradients per damping family, as a line calibration runs it
        _synth("fit_center", lam=1560.0, N=25007, L=120000, step="fit", eta=1e-3, fam=True),
        # the instrument operator on one spectrum and its VJP, with rotation, APOGEE-like pixels
        dict(kind="inst", name="instrument", N=37550, rot=True),
        # one evaluation of the calibration objective: two stars, three spectra, 42,886 records
        dict(kind="cal", name="calibration", N=37550, records=42886, n_bands=30),
        # independent stars of unlike windows and line counts, spectra and gradients in one batch
        dict(kind="batch", name="batch", stars=8, n_max=37550, l_max=200000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["synth"] * 7 + ["inst", "cal", "batch"])
    if kind == "inst":
        return dict(kind="inst", N=_log(rng, 30000, 37550), rot=rng.random() < 0.5)
    if kind == "cal":
        return dict(kind="cal", N=_log(rng, 6000, 37550), records=_log(rng, 2000, 42886), n_bands=rng.randint(1, 30))
    if kind == "batch":
        return dict(kind="batch", stars=rng.randint(2, 8), n_max=_log(rng, 8000, 37550), l_max=_log(rng, 20000, 200000))
    lam = rng.uniform(350.0, 1600.0)
    N = _log(rng, 900, 37550)
    per_px = math.exp(rng.uniform(math.log(0.5), math.log(8.0)))        # lines per pixel
    c = dict(SYNTH, lam=round(lam, 2), N=N, L=max(300, int(per_px * N * min(1.0, lam / 1500.0))), S=rng.randint(3, 40),
             D=rng.choice([72, 72, 72, 80, 64, 56, rng.randint(33, 80)]), teff=round(rng.uniform(3500.0, 7000.0), 1),
             logg=round(rng.uniform(1.0, 5.0), 2), xi=round(rng.uniform(0.5, 2.5), 2), bands=rng.choice([0.0, 0.3]),
             step=rng.choice(["fwd", "fit", "fit", "autograd"]), tile=rng.choice([0, 0, 0, 32]))
    kind = rng.choice(["plain", "plain", "plain", "e2", "scatter", "center", "fam"])
    if kind == "e2":
        c["quad"] = "e2"
    elif kind == "scatter":
        c["sigma_c"] = round(rng.uniform(0.2, 1.0), 2)
    elif kind in ("center", "fam"):
        c["eta"] = 1e-3 if kind == "center" else 0.0
        c["fam"] = c["step"] == "fit"
    return c


# ----------------------------------------------------------------------- inputs
def _atmosphere(rng, teff, logg, S, D, n_mol, lam_ref, feh=0.0, sigma_c=0.0):
    m = 10.0 ** (-3.0 + 4.0 * np.arange(D) / (D - 1))
    T = teff * (0.75 * (m + 2.0 / 3.0)) ** 0.25                          # grey
    scale = 10.0 ** logg / (1.1 * KB * teff)
    nH = scale * m
    mass = rng.uniform(12.0, 60.0, S)
    logA = rng.uniform(-8.0, -4.0, S) + feh
    chi = rng.uniform(5.0, 9.0, S)
    U = rng.integers(1, 11, size=(S, 2)).astype(np.float64)
    if n_mol:
        mass[S - n_mol:] = [26.0, 28.0][:n_mol]
        chi[S - n_mol:] = np.inf
    return NS(T=T, m=m, ne=1e-4 * scale * m ** 0.8, npert=nH, rho=1.4 * AMU * nH,
              n_species=(10.0 ** logA)[:, None] * nH[None, :], chi_ion_eV=chi,
              U=np.repeat(U[:, :, None], D, axis=2), mass_amu=mass, kappa0=1.0, lam_ref_nm=lam_ref, alpha=-1.0,
              sigma_c=np.full(D, sigma_c) if sigma_c else None, sigma_alpha=0.0, D=D, S=S)


def _lines(rng, L, lam_lo, lam_hi, S, n_mol, bands):
    """Atomic lines, a share of them replaced by regularly spaced molecular band sequences."""
    n_band = int(bands * L / 600.0) * 600 if n_mol else 0
    nb = n_band // 600
    lam = rng.uniform(lam_lo, lam_hi, L)
    loggf = rng.uniform(-4.0, 0.0, L)
    E = rng.uniform(0.0, 6.0, L)
    sp = rng.integers(0, S - n_mol, L).astype(np.int32)
    ion = rng.integers(0, 2, L).astype(np.int32)
    if n_band:
        d = rng.uniform(0.01, 0.05, nb)
        d = np.minimum(d, 0.999 * (lam_hi - lam_lo) / 600.0)
        head = lam_lo + rng.random(nb) * (lam_hi - lam_lo - d * 599)
        lam[:n_band] = (head[:, None] + d[:, None] * np.arange(600)).ravel()
        loggf[:n_band] = rng.normal(-2.0, 1.0, n_band)
        E[:n_band] = rng.uniform(0.0, 2.0, n_band)
        sp[:n_band] = np.repeat(rng.integers(S - n_mol, S, nb), 600)
        ion[:n_band] = 0
    return NS(lam0_nm=lam, loggf=loggf, E_eV=E, species=sp, ion=ion, log_grad=rng.uniform(7.0, 9.0, L),
              log_gstark=rng.uniform(-7.0, -4.0, L), log_gvdw=rng.uniform(-9.0, -7.0, L), L=L)


def _grid(lam, N):
    return NS(lam_first_nm=float(lam), R=R_GRID, N=int(N))


def _lam(g):
    return g.lam_first_nm * (1.0 + 1.0 / g.R) ** np.arange(g.N, dtype=np.float64)


def _target(rng, N):
    """An observed normalised spectrum: absorption of random depth, noise SIGMA."""
    return (1.0 - 0.8 * rng.random(N) ** 2 + rng.normal(0.0, SIGMA, N)).astype(np.float32)


def _workload(rng, c):
    n_mol = 2 if c["bands"] else 0
    g = _grid(c["lam"], c["N"])
    hi = c["lam"] * (1.0 + 1.0 / R_GRID) ** (c["N"] - 1)
    atm = _atmosphere(rng, c["teff"], c["logg"], c["S"], c["D"], n_mol, math.sqrt(c["lam"] * hi), c.get("feh", 0.0),
                      c.get("sigma_c", 0.0))
    ln = _lines(rng, c["L"], c["lam"], hi, c["S"], n_mol, c["bands"])
    big = c["L"] > 1000000
    f = lambda n, s: np.zeros(n, np.float32) if big else rng.normal(0.0, s, n).astype(np.float32)  # noqa: E731
    par = NS(dgf=f(ln.L, 0.05), ddamp=f(ln.L, 0.1), dA=f(c["S"], 0.05), xi_kms=np.float32(c["xi"]),
             ddamp_family=np.stack([f(ln.L, 0.1) for _ in range(3)]) if c.get("fam") else None)
    return NS(grid=g, lines=ln, atm=atm, params=par, window_nm=W_NM, quadrature=c.get("quad", "gauss3"),
              center_eta=c.get("eta", 0.0)), _target(rng, g.N)


def _rng(seed):
    return np.random.Generator(np.random.PCG64([seed, 24141]))


def _inputs(c, seed):
    return _workload(_rng(seed), c)


def _stars(c, seed):
    """Stars of a batch: window and line count drawn per star (the case's own), the rest from the seed."""
    out, size = [], _rng(0)
    for b in range(c["stars"]):
        rng = np.random.Generator(np.random.PCG64([seed, 24142, b]))
        N = min(int(size.integers(5000, 40001)), c["n_max"])
        i0 = int(size.integers(0, 37550 - N + 1))
        out.append(_workload(rng, dict(lam=1500.0 * (1.0 + 1.0 / R_GRID) ** i0, N=N,
                                       L=int(size.integers(10000, c["l_max"] + 1)), S=20, D=72,
                                       teff=rng.uniform(3500.0, 7000.0), logg=rng.uniform(1.0, 5.0),
                                       feh=rng.uniform(-2.0, 0.5), xi=rng.uniform(0.5, 2.5), bands=0.3)))
    return out


def _spectrum_like(rng, N):
    """A total and a continuum flux: smooth continuum, lines of a few pixels' width."""
    Fc = 1.0e6 * (1.0 + 0.3 * np.cos(np.arange(N) / N * 3.0 + rng.uniform(0, 6)))
    tau = np.zeros(N)
    at = rng.integers(0, N, N // 30)
    k = np.arange(-20, 21)
    depth, width = rng.exponential(0.6, at.size), rng.uniform(2.0, 5.0, at.size)
    np.add.at(tau, np.clip(at[:, None] + k, 0, N - 1), depth[:, None] * np.exp(-0.5 * (k / width[:, None]) ** 2))
    return (Fc * np.exp(-tau)).astype(np.float32), Fc.astype(np.float32)


def _apogee(g):
    """Log-uniform observed pixels (6e-6 dex) in three detector ranges, LSF of resolving power 20,000-25,000."""
    x0, x1 = math.log(g.lam_first_nm) + 1e-3, math.log(g.lam_first_nm) + (g.N - 1) * math.log1p(1.0 / g.R) - 1e-3
    lam = np.exp(np.arange(x0, x1, 6.0e-6 * LN10))
    lam = lam[~(((lam > 1581.0) & (lam < 1585.0)) | ((lam > 1644.0) & (lam < 1647.0)))]
    return lam, 1.0 / (2.0 * math.sqrt(2.0 * math.log(2.0)) * (20000.0 + 5000.0 * (lam - lam[0]) / (lam[-1] - lam[0])))


def _inst_inputs(c, seed):
    rng = _rng(seed)
    g = _grid(1500.0, c["N"])
    F, Fc = _spectrum_like(rng, g.N)
    lam, sig = _apogee(g)
    vel = [rng.uniform(-30.0, 30.0), rng.uniform(1.0, 15.0)] + ([rng.uniform(5.0, 38.0)] if c["rot"] else [])
    df = rng.normal(0.0, 1.0, lam.size).astype(np.float32) + np.float32(0.5)
    return NS(grid=g, F=F, Fc=Fc, lam=lam, sig=sig, vel=np.array(vel, np.float32), df=df, vb_max=20.0,
              vrot_max=40.0 if c["rot"] else 0.0, eps=0.6)


def _cal_inputs(c, seed):
    """A solar standard and a giant observed at two epochs, sharing one line list of
    records in complexes (calibrated) and molecular bands (held fixed).  The records'
    wavelengths, energies and strengths are the catalogue's, the same for every seed."""
    seeded, rng = _rng(seed), _rng(0)
    g = _grid(1500.0, c["N"])
    lo, hi = 1500.0, 1500.0 * (1.0 + 1.0 / R_GRID) ** (g.N - 1)
    n = c["records"]
    cid = np.repeat(np.arange(n), 1 + rng.poisson(0.7, n))[:n]
    k = int(cid[-1]) + 1
    rec = _lines(rng, n, lo, hi, 18, 0, 0.0)
    rec.lam0_nm = rng.uniform(lo, hi, k)[cid] + rng.uniform(-0.012, 0.012, n)
    rec.E_eV = np.maximum(rng.uniform(0.0, 6.0, k)[cid] + rng.uniform(-0.7, 0.7, n) * 1.239841984e-4, 0.0)
    rec.loggf = rng.uniform(-4.0, 0.0, k)[cid] + rng.normal(0.0, 0.3, n)
    rec.species = rng.integers(0, 18, k).astype(np.int32)[cid]
    rec.ion = rng.integers(0, 2, k).astype(np.int32)[cid]
    rng = seeded
    mol = _lines(rng, 600 * c["n_bands"], lo, hi, 20, 2, 1.0)
    ln = NS(**{f: np.concatenate([getattr(rec, f), getattr(mol, f)]) for f in
               ("lam0_nm", "loggf", "E_eV", "species", "ion", "log_grad", "log_gstark", "log_gvdw")})
    ln.L = ln.lam0_nm.size
    std, ys, sp_seed = [], [], int(rng.integers(1 << 30))
    for teff, logg, feh, xi, vb, n_ep, step in ((5777.0, 4.44, 0.0, 0.7, 1.55, 1, 1.5), (4286.0, 1.66, -0.52, 1.7, 2.5, 2, 1.4)):
        atm = _atmosphere(_rng(sp_seed), teff, logg, 20, 72, 2, math.sqrt(lo * hi), feh)
        wl = NS(grid=g, lines=ln, atm=atm, window_nm=W_NM, quadrature="gauss3", center_eta=0.0,
                params=NS(dgf=None, ddamp=None, dA=np.zeros(20, np.float32), xi_kms=xi, ddamp_family=None))
        lam = np.exp(math.log(lo) + math.log1p(1.0 / g.R) * np.arange(60, g.N - 61, step))
        for e in range(n_ep):
            w = np.where(rng.random(lam.size) < 0.1, 0.0, rng.uniform(0.5, 1.0, lam.size)).astype(np.float32)
            std.append(NS(name="s%d" % len(std), wl=wl, lam_obs_nm=lam, lsf_sigma_ln=np.full(lam.size, 1.0 / (2.3548 * 2.5e5)),
                          vb_max_kms=3.0, vel=(0.0, vb), w=w, c=1.0 / (2 * n_ep * float(w.sum()))))
            ys.append(_target(rng, lam.size))
    active = np.arange(ln.L) < n
    return NS(cal=NS(grid=g, lines=ln, active=active, standards=std), ys=ys,
              draw=lambda G: np.stack([rng.normal(0.0, s, G) for s in (0.1, 0.3, 0.3, 0.2)]).astype(np.float32))


# ------------------------------------------------------------------- the passes
def _fit_buffers(plan, fam):
    e = lambda *n: torch.empty(n, device="cuda")  # noqa: E731
    star = e(plan.S + 1)                            # the star's own parameters: abundances, microturbulence
    return NS(F=e(plan.N), Fc=e(plan.N), dF=e(plan.N), loss=e(1), gf=e(plan.L),
              damp=e(3, plan.L) if fam else e(plan.L), star=star, A=star[:-1], xi=star[-1:])


def _plan(wl, c):
    return pz.plan_for(wl, tile_px=c.get("tile", 0), flags=pz.PZ_FLAG_DAMPING_FAMILIES if c.get("fam") else 0)


def prepare(case, seed):
    c, kind = case, case["kind"]
    dev = lambda a: torch.as_tensor(a, device="cuda")  # noqa: E731
    if kind == "synth":
        wl, y = _inputs(c, seed)
        s = NS(kind=c["step"], plan=_plan(wl, c), atm=pz.Atmos(wl.atm), y=dev(y))
        s.b = _fit_buffers(s.plan, c["fam"])
        if c["step"] == "autograd":
            p = wl.params
            s.leaves = [dev(np.atleast_1d(a)).requires_grad_() for a in (p.dgf, p.ddamp, p.dA, p.xi_kms)]
        else:
            s.par = pz.Params.from_host(wl.params)
        return s
    if kind == "batch":
        keep, stars = [], []
        for wl, y in _stars(c, seed):
            k = NS(plan=_plan(wl, c), atm=pz.Atmos(wl.atm), par=pz.Params.from_host(wl.params), y=dev(y))
            k.b = _fit_buffers(k.plan, False)
            keep.append(k)
            p = lambda t: t.data_ptr()  # noqa: E731
            stars.append(pz.pz_star(k.plan.handle, k.atm.c, k.par.c, p(k.b.F), p(k.b.Fc), None, p(k.y), SIGMA, p(k.b.loss),
                                    p(k.b.gf), p(k.b.damp), p(k.b.A), p(k.b.xi)))
        return NS(kind="batch", keep=keep, batch=pz.Batch(stars))
    if kind == "inst":
        i = _inst_inputs(c, seed)
        inst = pz.Instrument(i.grid, i.lam, i.sig, i.vb_max, vrot_max_kms=i.vrot_max, limb_eps=i.eps)
        e = lambda n: torch.empty(n, device="cuda")  # noqa: E731
        return NS(kind="inst", inst=inst, F=dev(i.F), Fc=dev(i.Fc), vel=dev(i.vel), df=dev(i.df), f=e(inst.P), dF=e(inst.N),
                  dFc=e(inst.N), g=e(inst.n_vel))
    from paper_2607_24141_amd import calibrate
    i = _cal_inputs(c, seed)
    cal = calibrate.Calibration(i.cal, i.ys)
    return NS(kind="cal", cal=cal, theta=dev(i.draw(cal.G)))


def run(state):
    s = state
    if s.kind == "fwd":
        pz.synth_forward(s.plan, s.atm, s.par, s.b.F, s.b.Fc)
        return dict(F=s.b.F, Fc=s.b.Fc)
    if s.kind == "fit":
        b = s.b
        pz.synth_forward(s.plan, s.atm, s.par, b.F, b.Fc)
        pz.pz_chi2_seed(b.F, b.Fc, s.y, SIGMA, b.dF, loss=b.loss)
        pz.synth_backward(s.plan, s.atm, s.par, b.dF, b.gf, b.damp, b.A, b.xi)
        return dict(F=b.F, Fc=b.Fc, loss=b.loss, gf=b.gf, damp=b.damp, star=b.star)
    if s.kind == "autograd":
        F, Fc = pz.PzSynth().apply(s.plan, s.atm, *s.leaves)
        loss = (((F / Fc - s.y) / SIGMA) ** 2).sum()
        g = torch.autograd.grad(loss, s.leaves)
        return dict(F=F.detach(), Fc=Fc, loss=loss.detach(), gf=g[0], damp=g[1], star=torch.cat([g[2], g[3]]))
    if s.kind == "batch":
        pz.synth_batch(s.batch, pz.PZ_MODE_FWD_BWD)
        return [dict(F=k.b.F, Fc=k.b.Fc, loss=k.b.loss, gf=k.b.gf, damp=k.b.damp, star=k.b.star) for k in s.keep]
    if s.kind == "inst":
        pz.pz_inst_forward(s.inst, s.F, s.Fc, s.vel, f=s.f)
        pz.pz_inst_backward(s.inst, s.F, s.Fc, s.vel, s.df, s.dF, s.dFc, s.g)
        return dict(f=s.f, dF=s.dF, dFc=s.dFc, vel=s.g)
    loss, grad = s.cal.evaluate(s.theta)
    return dict(loss=loss, grad=grad)


# ------------------------------------------------------------------------- work
def _evals(lam, N, L, D):
    """Voigt evaluations of uniform lines: pixels within W of a line, at every depth."""
    mid = lam * math.exp(0.5 * N / R_GRID)
    return L * D * min(N, 2.0 * W_NM / (mid / R_GRID))


def _synth_work(lam, N, L, S, D, grad):
    # 20 operations per evaluation is the least of the Voigt forms in use (a far-wing term and its detuning);
    # a gradient evaluates the function and two derivatives
    ev = _evals(lam, N, L, D)
    return (L * 72.0 + N * 8.0 + (2.0 * L * 4.0 + N * 8.0 if grad else 0.0) + 8.0 * D * (3 * S + 5), ev * (20.0 + (30.0 if grad else 0.0)))


def work(case):
    c, kind = case, case["kind"]
    if kind == "synth":
        b, f = _synth_work(c["lam"], c["N"], c["L"], c["S"], c["D"], c["step"] != "fwd")
    elif kind == "batch":
        # the mean star of the drawn windows (5,000 to n_max pixels) and line counts (10,000 to l_max)
        b, f = _synth_work(1600.0, 0.5 * (5000 + c["n_max"]), 0.5 * (10000 + c["l_max"]), 20, 72, True)
        b, f = b * c["stars"], f * c["stars"]
    elif kind == "inst":
        P, N = c["N"] * 0.22, c["N"]
        taps = 2 * (2 * 81 + (2 * 41 if c["rot"] else 0))
        b, f = N * 16.0 + P * 24.0, 3.0 * N * taps * 2.0
    else:
        L = c["records"] + 600 * c["n_bands"]
        b, f = _synth_work(1600.0, c["N"], L, 20, 72, True)
        b, f = 2 * b + c["records"] * 32.0, 2 * f
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------------ exact
def _weideman(n):
    """Coefficients of Weideman's n-term expansion of w(z)."""
    M = 4 * n
    k = np.arange(-M + 1, M)
    L = math.sqrt(n / math.sqrt(2.0))
    t = L * np.tan(k * math.pi / M / 2.0)
    f = np.concatenate([[0.0], np.exp(-t * t) * (L * L + t * t)])
    a = np.real(np.fft.fft(np.fft.fftshift(f))) / (2 * M)
    return L, a[1:n + 1][::-1].copy()


_WL, _WA = _weideman(56)


def _faddeeva(v, a):
    """w(v + i a), a > 0: continued fraction where |z| >= 8, else Weideman's expansion."""
    z = torch.complex(v, a)
    w = torch.empty_like(z)
    far = (v * v + a * a) >= 64.0
    zf = z[far]
    r = zf
    for k in range(16, 0, -1):
        r = zf - (0.5 * k) / r
    w[far] = (1j / math.sqrt(math.pi)) / r
    zn = z[~far]
    if zn.numel():
        iz = 1j * zn
        d = 1.0 / (_WL - iz)
        Z = (_WL + iz) * d
        p = torch.full_like(Z, _WA[0])
        for c in _WA[1:]:
            p = p * Z + c
        w[~far] = (2.0 * p * d + 1.0 / math.sqrt(math.pi)) * d
    return w


class _Exact:
    """The synthesis of one workload in float64 (device tensors)."""

    def __init__(self, wl, par=None):
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        t = lambda a: torch.as_tensor(np.asarray(a, np.float64), device=self.dev)  # noqa: E731
        self.wl, self.t = wl, t
        atm, ln, g = wl.atm, wl.lines, wl.grid
        par = par or wl.params
        lam = _lam(g)
        self.lam = t(lam)
        order = np.argsort(ln.lam0_nm, kind="stable")
        self.order = torch.as_tensor(order, device=self.dev)
        l0 = ln.lam0_nm[order]
        lo = np.clip(np.searchsorted(lam, l0 - W_NM) - 1, 0, g.N)
        for _ in range(2):
            lo = np.where((lo < g.N) & ~(np.abs(lam[np.minimum(lo, g.N - 1)] - l0) <= W_NM) & (lam[np.minimum(lo, g.N - 1)] < l0), lo + 1, lo)
        hi = np.clip(np.searchsorted(lam, l0 + W_NM), -1, g.N - 1)
        for _ in range(2):
            hi = np.where((hi >= 0) & ~(np.abs(lam[np.maximum(hi, 0)] - l0) <= W_NM) & (lam[np.maximum(hi, 0)] > l0), hi - 1, hi)
        self.lo, self.hi = torch.as_tensor(lo, device=self.dev), torch.as_tensor(hi, device=self.dev)
        T, m = t(atm.T), t(atm.m)
        self.T, self.m = T, m
        # populations (two-stage Saha)
        chi, U = t(atm.chi_ion_eV)[:, None] * EV, t(atm.U)
        phi = 2.0 * U[:, 1] / U[:, 0] * (2.0 * math.pi * ME * KB / H ** 2) ** 1.5 * T ** 1.5 * torch.exp(-chi / (KB * T)) / t(atm.ne)
        phi = torch.where(torch.isfinite(chi), phi, torch.zeros_like(phi))
        fr = torch.stack([1.0 / (1.0 + phi), phi / (1.0 + phi)], 1)
        zero = np.zeros(ln.L)
        pick = lambda a: t(zero if a is None else a)[self.order]  # noqa: E731
        dA = t(par.dA)
        pop = (10.0 ** dA)[:, None, None] * t(atm.n_species)[:, None, :] * fr / (t(atm.rho) * U)
        self.sp = torch.as_tensor(ln.species.astype(np.int64), device=self.dev)[self.order]
        ion = torch.as_tensor(ln.ion.astype(np.int64), device=self.dev)[self.order]
        self.xi = float(np.float32(par.xi_kms)) * 1e5
        self.dv = torch.sqrt(2.0 * KB * T / (t(atm.mass_amu)[:, None] * AMU) + self.xi ** 2)
        self.l0 = t(l0)
        lc = self.l0 * 1e-7
        fam = par.ddamp_family
        fam = [None] * 3 if fam is None else fam
        sc = 10.0 ** pick(par.ddamp)
        gam = [10.0 ** (pick(q) + pick(d)) * sc for q, d in zip((ln.log_grad, ln.log_gstark, ln.log_gvdw), fam)]
        gf = 10.0 ** (pick(ln.loggf) + pick(par.dgf))
        E = pick(ln.E_eV) * EV
        ne, npt = t(atm.ne), t(atm.npert)

        def params(b):                               # per (line of the block, depth)
            dv = self.dv[self.sp[b]]
            G = [gam[0][b][:, None].expand_as(dv), gam[1][b][:, None] * ne, gam[2][b][:, None] * npt]
            Gt = G[0] + G[1] + G[2]
            a = Gt * lc[b][:, None] / (4.0 * math.pi * dv)
            K = (math.pi * QE ** 2 / (ME * C)) * pop[self.sp[b], ion[b]] * gf[b][:, None] * torch.exp(-E[b][:, None] / (KB * T)) * \
                -torch.expm1(-H * C / (lc[b][:, None] * KB * T)) * lc[b][:, None] / (math.sqrt(math.pi) * dv)
            V = None
            if wl.center_eta:
                eta = wl.center_eta
                Rr = K / (atm.kappa0 * (self.l0[b][:, None] / atm.lam_ref_nm) ** atm.alpha)
                V = torch.maximum(torch.sqrt(torch.clamp(torch.log(Rr / eta), min=0.0)), torch.sqrt(a * Rr / (math.sqrt(math.pi) * eta)))
                V = torch.where(Rr * torch.special.erfcx(a) >= eta, V, torch.full_like(V, -1.0))
            return dv, a, K, V, G, Gt

        self.params = params
        self.kc = atm.kappa0 * (self.lam / atm.lam_ref_nm) ** atm.alpha
        lcm = self.lam[None, :] * 1e-7
        self.B = 2.0 * H * C * C / lcm ** 5 / torch.expm1(H * C / (lcm * KB * T[:, None])) * 1e-7

    def blocks(self):
        """(line block, pixel of each line, in window, v [lines, D], line-depth parameters) over all window offsets."""
        L, D = self.l0.numel(), self.T.numel()
        step = max(1, 4_000_000 // D)
        for b0 in range(0, L, step):
            b = slice(b0, min(L, b0 + step))
            p = self.params(b)
            lo, hi = self.lo[b], self.hi[b]
            for k in range(int((hi - lo).max().clamp(min=-1)) + 1):
                px = lo + k
                inw = px <= hi
                px = torch.where(inw, px, torch.zeros_like(px))
                x = self.l0[b] / self.lam[px] - 1.0
                v = x[:, None] * C / p[0]
                keep = inw[:, None].expand_as(v) if p[3] is None else inw[:, None] & (v.abs() <= p[3])
                yield b, px, keep, v, p

    def kappa(self):
        kap = torch.zeros(self.lam.numel(), self.T.numel(), dtype=torch.float64, device=self.dev)
        for b, px, keep, v, (dv, a, K, V, G, Gt) in self.blocks():
            kap.index_add_(0, px, torch.where(keep, K * _faddeeva(v, a).real, torch.zeros_like(v)))
        return kap.t().contiguous()

    def line_grads(self, g):
        """Gradients per line (catalogue order), species and microturbulence for g = dL/dkappa [D, N]."""
        gt = g.t().contiguous()
        L = self.l0.numel()
        z = lambda *n: torch.zeros(n, dtype=torch.float64, device=self.dev)  # noqa: E731
        gf, fam, xi = z(L), z(3, L), z(1)
        for b, px, keep, v, (dv, a, K, V, G, Gt) in self.blocks():
            w = _faddeeva(v, a)
            Hr, Li = w.real, w.imag
            Ha, Hv = 2.0 * (v * Li + a * Hr) - 2.0 / math.sqrt(math.pi), -2.0 * (v * Hr - a * Li)
            gK = torch.where(keep, gt[px] * K, torch.zeros_like(v))
            gf[b] += LN10 * (gK * Hr).sum(1)
            d = LN10 * gK * a * Ha / Gt
            for f in range(3):
                fam[f][b] += (d * G[f]).sum(1)
            xi += (-gK * (Hr + a * Ha + v * Hv) * (self.xi / dv ** 2 * 1e5)).sum()
        A = z(self.wl.atm.S).index_add_(0, self.sp, gf)
        back = lambda q: torch.empty_like(q).index_copy_(-1, self.order, q)  # noqa: E731
        return back(gf), back(fam), A, xi

    def transfer(self, kap):
        """Both fluxes, kap [D, N] the line opacity."""
        kc = self.kc[None, :].expand_as(kap)
        if self.wl.atm.sigma_c is None:
            return _flux(self.B, _tau(kc + kap, self.m), self.wl.quadrature), _flux(self.B, _tau(kc, self.m), self.wl.quadrature)
        sig = self.t(self.wl.atm.sigma_c)[:, None]
        out = []
        for ka in (kc + kap, kc):
            chi = ka + sig
            out.append(_Scatter.apply(_tau(chi, self.m), ka / chi, self.B))
        return out


def _tau(chi, m):
    t = [chi[0] * m[0]]
    for j in range(1, chi.shape[0]):
        t.append(t[-1] + 0.5 * (chi[j - 1] + chi[j]) * (m[j] - m[j - 1]))
    return torch.stack(t)


def _segment(x):
    """exp(-x) and (1 - (1 + x) exp(-x)) / x."""
    e = torch.exp(-x)
    xs, xl = torch.clamp(x, max=0.05), torch.clamp(x, min=0.05)
    s = torch.zeros_like(x)
    for n in range(12, 1, -1):
        s = s + (-1.0) ** n * (n - 1) * xs ** (n - 1) / math.factorial(n)
    return e, torch.where(x < 0.05, s, (1.0 - (1.0 + xl) * torch.exp(-xl)) / xl)


def _surface(S, tau):
    return S[0] - tau[0] * (S[1] - S[0]) / (tau[1] - tau[0])


def _outward(S, tau, mu):
    """I+ at every depth (deepest first in the recurrence) and at the surface."""
    D = S.shape[0]
    Is = [S[D - 1] + mu * (S[D - 1] - S[D - 2]) / (tau[D - 1] - tau[D - 2])]
    e, lw = _segment((tau[1:] - tau[:-1]) / mu)
    for j in range(D - 2, -1, -1):
        Is.append(Is[-1] * e[j] + S[j] * (1.0 - e[j]) + (S[j + 1] - S[j]) * lw[j])
    e, lw = _segment(tau[0] / mu)
    St = _surface(S, tau)
    return torch.stack(Is[::-1]), Is[-1] * e + St * (1.0 - e) + (S[0] - St) * lw


def _inward(S, tau, mu):
    D = S.shape[0]
    e, lw = _segment(tau[0] / mu)
    Is = [S[0] * (1.0 - e) + (_surface(S, tau) - S[0]) * lw]
    e, lw = _segment((tau[1:] - tau[:-1]) / mu)
    for j in range(1, D):
        Is.append(Is[-1] * e[j - 1] + S[j] * (1.0 - e[j - 1]) + (S[j - 1] - S[j]) * lw[j - 1])
    return torch.stack(Is)


_G3 = [(0.5 - 0.5 * math.sqrt(0.6), 5.0 / 18.0), (0.5, 8.0 / 18.0), (0.5 + 0.5 * math.sqrt(0.6), 5.0 / 18.0)]


def _angles(quad):
    if quad == "gauss3":
        return _G3
    # the exact angle integral: Gauss-Legendre in u with mu = u^3, which clusters nodes at mu = 0
    x, w = np.polynomial.legendre.leggauss(96)
    u = 0.5 * (x + 1.0)
    return list(zip(u ** 3, 0.5 * w * 3.0 * u * u))


def _flux(S, tau, quad):
    F = 0.0
    for mu, w in _angles(quad):
        F = F + 2.0 * math.pi * w * mu * _outward(S, tau, mu)[1]
    return F


class _Scatter(torch.autograd.Function):
    """Flux of S = eps B + (1 - eps) Lambda S, solved by iteration; gradients at the fixed point."""

    @staticmethod
    def step(S, tau, eps, B):
        J = 0.0
        for mu, w in _G3:
            J = J + 0.5 * w * (_outward(S, tau, mu)[0] + _inward(S, tau, mu))
        return eps * B + (1.0 - eps) * J

    @staticmethod
    def forward(ctx, tau, eps, B):
        S = B.clone()
        for _ in range(400):
            Sn = _Scatter.step(S, tau, eps, B)
            d = float(((Sn - S).abs() / Sn).max())
            S = Sn
            if d < 1e-14:
                break
        ctx.save_for_backward(tau, eps, B, S)
        return _flux(S, tau, "gauss3")

    @staticmethod
    def backward(ctx, gF):
        tau, eps, B, S = ctx.saved_tensors
        with torch.enable_grad():
            tau, eps, S = (q.detach().requires_grad_() for q in (tau, eps, S))
            gS, gt = torch.autograd.grad(_flux(S, tau, "gauss3"), (S, tau), gF)
            S1 = _Scatter.step(S, tau, eps, B)
            lam = gS
            for _ in range(400):
                ln = gS + torch.autograd.grad(S1, S, lam, retain_graph=True)[0]
                d = float((ln - lam).abs().max() / ln.abs().max())
                lam = ln
                if d < 1e-14:
                    break
            t2, ge = torch.autograd.grad(S1, (tau, eps), lam)
        return gt + t2, ge, None


def _exact_fit(wl, y, fam):
    ex = _Exact(wl)
    kap = ex.kappa().requires_grad_()
    F, Fc = ex.transfer(kap)
    loss = (((F / Fc - ex.t(y)) / SIGMA) ** 2).sum()
    g, = torch.autograd.grad(loss, kap)
    gf, gfam, A, xi = ex.line_grads(g)
    d = lambda q: q.detach()  # noqa: E731
    return dict(F=d(F), Fc=d(Fc), loss=d(loss).reshape(1), gf=gf, damp=gfam if fam else gfam.sum(0), star=torch.cat([A, xi]))


def _shifted(G, k):
    """G_{i-k} where it exists, else 0."""
    N = G.shape[-1]
    z = torch.zeros_like(G)
    if k >= 0:
        z[..., k:] = G[..., :N - k]
    else:
        z[..., :N + k] = G[..., -k:]
    return z


class _Convolve(torch.autograd.Function):
    """(T G)_i = sum_k w_|k| G_{i-k} / Z_i over the pixels that exist, with dw/ds for one width s."""

    @staticmethod
    def forward(ctx, G, s, w, dw):
        one = torch.ones_like(G[0])
        num, dnum, Z, dZ = torch.zeros_like(G), torch.zeros_like(G), torch.zeros_like(one), torch.zeros_like(one)
        for k in range(-len(w) + 1, len(w)):
            g, o = _shifted(G, k), _shifted(one, k)
            num += w[abs(k)] * g
            dnum += dw[abs(k)] * g
            Z += w[abs(k)] * o
            dZ += dw[abs(k)] * o
        ctx.save_for_backward((dnum * Z - num * dZ) / Z ** 2, Z)
        ctx.w = w
        return num / Z

    @staticmethod
    def backward(ctx, g):
        dT, Z = ctx.saved_tensors
        q, out = g / Z, torch.zeros_like(g)
        for k in range(-len(ctx.w) + 1, len(ctx.w)):
            out += ctx.w[abs(k)] * _shifted(q, -k)
        return out, (g * dT).sum(), None, None


def _rot_taps(s, JR, eps):
    cdf = lambda y: ((1 - eps) * (y * np.sqrt(np.maximum(1 - y * y, 0)) + np.arcsin(y)) + 0.5 * math.pi * eps * (y - y ** 3 / 3)) / (math.pi * (1 - eps / 3))  # noqa: E731
    pdf = lambda y: (2 * (1 - eps) * np.sqrt(np.maximum(1 - y * y, 0)) + 0.5 * math.pi * eps * (1 - y * y)) / (math.pi * (1 - eps / 3))  # noqa: E731
    b = (np.arange(JR + 2) - 0.5) / s
    c = cdf(np.clip(b, -1, 1))
    d = np.where(np.abs(b) < 1, pdf(np.clip(b, -1, 1)) * (-b / s), 0.0)
    return c[1:] - c[:-1], d[1:] - d[:-1]


def _observe(g, lam_obs, sig, vb_max, vrot_max, eps, F2, vel):
    """K S R B of both fluxes F2 [2, N] for velocities vel (a tensor that may need a gradient)."""
    h = math.log1p(1.0 / g.R)
    dev, N = F2.device, g.N
    s = vel[1] / (C_KMS * h)
    J = int(math.ceil(4.0 * vb_max / C_KMS / h))
    k = np.arange(J + 1)
    sf = float(s)
    w = np.exp(-0.5 * (k / sf) ** 2)
    G = _Convolve.apply(F2, s, w, w * k * k / sf ** 3)
    if vrot_max > 0:
        s = vel[2] / (C_KMS * h)
        G = _Convolve.apply(G, s, *_rot_taps(float(s), int(math.ceil(vrot_max / C_KMS / h + 0.5)), eps))
    t = torch.log1p(vel[0] / C_KMS) / h
    m = math.floor(-float(t))
    r = -t - m
    xp, x0 = np.log(lam_obs), math.log(g.lam_first_nm)
    lo = np.ceil((xp - 4.0 * sig - x0) / h).astype(np.int64)
    hi = np.floor((xp + 4.0 * sig - x0) / h).astype(np.int64)
    c, a = torch.as_tensor((xp - x0) / h, device=dev), torch.as_tensor(h * h / (2.0 * sig ** 2), device=dev)
    lo, hi = torch.as_tensor(lo, device=dev), torch.as_tensor(hi, device=dev)
    num, W = 0.0, 0.0
    for q in range(int((hi - lo).max()) + 1):
        i = lo + q
        wq = torch.where(i <= hi, torch.exp(-((i - c) ** 2) * a), torch.zeros_like(c))
        k0, k1 = (i + m).clamp(0, N - 1), (i + m + 1).clamp(0, N - 1)
        num = num + wq * ((1.0 - r) * G[:, k0] + r * G[:, k1])
        W = W + wq
    return num / W


def _exact_inst(c, seed):
    i = _inst_inputs(c, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    t = lambda a: torch.as_tensor(np.asarray(a, np.float64), device=dev)  # noqa: E731
    F2, vel = torch.stack([t(i.F), t(i.Fc)]).requires_grad_(), t(i.vel).requires_grad_()
    K = _observe(i.grid, i.lam, i.sig, i.vb_max, i.vrot_max, i.eps, F2, vel)
    f = K[0] / K[1]
    g, gv = torch.autograd.grad(f, (F2, vel), t(i.df))
    return dict(f=f.detach(), dF=g[0], dFc=g[1], vel=gv)


def _groups(cal):
    """Greedy groups: strongest line first, its ungrouped neighbours within 2 cm^-1 and 0.035 nm join it."""
    ln, n = cal.lines, int(cal.active.sum())
    q = np.full(ln.L, -1)
    key = ln.species[:n].astype(np.int64) * 2 + ln.ion[:n]
    by = np.lexsort((ln.lam0_nm[:n], key))
    pos = np.empty(n, np.int64)
    pos[by] = np.arange(n)
    G = 0
    for s in sorted(range(n), key=lambda i: (-ln.loggf[i], i)):
        if q[s] >= 0:
            continue
        for d in (1, -1):
            p = pos[s] if d == 1 else pos[s] - 1
            while 0 <= p < n and key[by[p]] == key[s] and abs(ln.lam0_nm[by[p]] - ln.lam0_nm[s]) <= 0.035:
                o = by[p]
                if q[o] < 0 and abs(ln.E_eV[o] - ln.E_eV[s]) <= 2.0 * 1.239841984e-4:
                    q[o] = G
                p += d
        G += 1
    return q, G


def _exact_cal(c, seed):
    i = _cal_inputs(c, seed)
    q, G = _groups(i.cal)
    theta = i.draw(G).astype(np.float64)
    X = np.where(q >= 0, theta[:, np.maximum(q, 0)], 0.0)
    loss, grad, by = 0.0, 0.0, {}
    for k, s in enumerate(i.cal.standards):
        by.setdefault(id(s.wl), []).append(k)
    for ks in by.values():
        wl = i.cal.standards[ks[0]].wl
        ex = _Exact(wl, NS(dgf=X[0], ddamp=None, dA=wl.params.dA, xi_kms=wl.params.xi_kms, ddamp_family=X[1:]))
        kap = ex.kappa().requires_grad_()
        F, Fc = ex.transfer(kap)
        part = 0.0
        for k in ks:
            s = i.cal.standards[k]
            K = _observe(wl.grid, s.lam_obs_nm, s.lsf_sigma_ln, s.vb_max_kms, 0.0, 0.6, torch.stack([F, Fc]), ex.t(np.float32(s.vel)))
            part = part + s.c * (ex.t(s.w) * (K[0] / K[1] - ex.t(i.ys[k])) ** 2).sum()
        g, = torch.autograd.grad(part, kap)
        gf, fam, _, _ = ex.line_grads(g)
        loss, grad = loss + part.detach(), grad + torch.cat([gf[None], fam])
    qt = torch.as_tensor(q, device=grad.device)
    out = torch.zeros(4, G, dtype=torch.float64, device=grad.device).index_add_(1, qt[qt >= 0], grad[:, qt >= 0])
    return dict(loss=loss.reshape(1), grad=out)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "inst":
        return _exact_inst(c, seed)
    if kind == "cal":
        return _exact_cal(c, seed)
    if kind == "batch":
        # the smallest stars in whole, as many as take a few seconds
        stars = _stars(c, seed)
        cost = [wl.lines.L for wl, _ in stars]
        take = [k for k in np.argsort(cost) if sum(q for q in cost if q <= cost[k]) <= 400000]
        return [_exact_fit(*stars[k], False) if k in take else None for k in range(len(stars))]
    if _evals(c["lam"], c["N"], c["L"], c["D"]) > 6e9:
        return None
    wl, y = _inputs(c, seed)
    if c["step"] != "fwd":
        r = _exact_fit(wl, y, c["fam"])
        return dict(r, loss=r["loss"][0]) if c["step"] == "autograd" else r
    ex = _Exact(wl)
    F, Fc = ex.transfer(ex.kappa())
    return dict(F=F, Fc=Fc)
