"""Damping ratios up to ten thousand with far pixels in the window, against the oracle."""
import numpy as np
import pytest

import workloads as W
from oracle import synth as O
from test_gpu_adjoint import gpu_vjp, grad_close_cond
from test_gpu_split import _kappa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a", [900.0, 2800.0, 7000.0])
def test_very_large_damping_ratios(gpu_lib, a):
    """A line whose damping ratio is a to 1.4 a over depth, with windows so
    wide that pixels lie beyond five times a: the far zone's polynomials in
    a^2 stay inside float32's range or the line has no far zone.  Opacities
    within and beyond its window, and its gradients.  The detuning's series
    (fourth order) loses up to 8e-7 at |x| = 0.1, twice that in the far
    opacity: 7e-6."""
    wl = W.tiny(seed=6, L=12, N=900, D=20, S=3, xi=0.0, lam_lo=500.0, R=3000.0, window_nm=50.0, Teff=3000.0)
    wl.atm.mass_amu[:] = 200.0
    wl.lines.lam0_nm[0] = 520.0
    wl.lines.log_gstark[0] = wl.lines.log_gvdw[0] = -30.0
    wl.lines.loggf[0] = 4.0
    p = wl.params
    dnu = O.line_depth_params(wl.atm, wl.lines, p.dgf, p.ddamp, p.dA, p.xi_kms)["dnu"]
    wl.lines.log_grad[0] = np.log10(a * 4.0 * np.pi * dnu[0].max())
    lp = O.line_depth_params(wl.atm, wl.lines, p.dgf, p.ddamp, p.dA, p.xi_kms)
    nu = O.C_LIGHT / (O.wavelengths_nm(wl.grid) * 1.0e-7)
    v = np.abs(nu - lp["nu_l"][0])[:, None] / lp["dnu"][0]
    inside = np.abs(O.wavelengths_nm(wl.grid) - 520.0) <= 50.0
    assert np.any(inside[:, None] & (v > 5.2 * lp["a"][0].max())) and not inside.all()
    np.testing.assert_allclose(_kappa(gpu_lib, wl), O.line_opacity(wl), rtol=7e-6, atol=1e-30)
    s = np.random.default_rng(6).normal(size=900).astype(np.float32)
    g = gpu_vjp(gpu_lib, wl, s)
    ref = O.adjoint(wl, p, s.astype(np.float64), conditions=True)
    grad_close_cond(g[0], ref["g_loggf"], ref["abs_loggf"], name="loggf")
    grad_close_cond(g[1], ref["g_damp"], ref["abs_damp"], name="damp")
