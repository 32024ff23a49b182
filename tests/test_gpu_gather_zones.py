"""The gather of the split line sums (near zone by direct evaluation, far zone
as a matrix product) against the direct gather and the oracle, at detunings
where the forms of the Voigt derivatives in use differ most."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import synth as O
from test_gpu_adjoint import gpu_vjp

pytestmark = pytest.mark.gpu


def _detunings(wl):
    """v [L, N, D] of every line at every pixel and depth (no window)."""
    p = wl.params
    lp = O.line_depth_params(wl.atm, wl.lines, p.dgf, p.ddamp, p.dA, p.xi_kms)
    nu = O.C_LIGHT / (O.wavelengths_nm(wl.grid) * 1.0e-7)
    return (nu[None, :, None] - lp["nu_l"][:, None, None]) / lp["dnu"][:, None, :]


def _dense(wl, seed=9):
    """The same workload with 2.2 lines per pixel of no strength (K = 0 in
    float32) added: a plan that takes the direct line sums."""
    n = int(2.2 * wl.grid.N)
    lam = O.wavelengths_nm(wl.grid)
    fill = W.atomic_lines(np.random.default_rng(seed), n, lam[0], lam[-1], wl.atm.S, loggf=np.full(n, -80.0))
    z = np.zeros(n)
    p = wl.params
    return W.Workload(wl.name + "+fill", wl.grid, wl.atm, W.concat_lines(wl.lines, fill),
                      W.Params(np.concatenate([p.dgf, z]), np.concatenate([p.ddamp, z]), p.dA, p.xi_kms), wl.window_nm)


@pytest.mark.parametrize("v0", [0.4, 0.92, 1.5, 3.0, 5.0])
def test_one_form_of_the_damping_derivative(gpu_lib, v0):
    """Damping gradients of weak lines from one pixel each, near |v| = v0: the
    split gather and the direct one evaluate the same form of a dH/da there and
    add its eight depths in the same order.  The lines are too weak for the
    opacity's rounding to show in dL/dkappa by more than one rounding: 2.4e-7
    of the sum of the terms' magnitudes, two units in the last place."""
    L = 20
    wl = W.tiny(seed=14, L=L, N=1500, D=8, S=4, xi=2.0, lam_lo=500.0, window_nm=0.05)
    lam = O.wavelengths_nm(wl.grid)
    wl.lines.lam0_nm[:] = lam[40 + 70 * np.arange(L)] * (1.0 + 1.0e-7 * np.arange(L))
    wl.lines.loggf[:] = -10.0
    v = np.abs(_detunings(wl)).mean(axis=2)
    s = np.zeros(wl.grid.N, np.float32)
    for k in range(L):                                    # windows do not overlap: one pixel for each line
        s[np.argmin(np.abs(v[k] - v0))] = 1.0
    assert np.all(O.line_opacity(wl) < 1e-3 * O.continuum_opacity(wl)[None, :])
    a, b = gpu_vjp(gpu_lib, wl, s), gpu_vjp(gpu_lib, _dense(wl), s)
    terms = O.adjoint(wl, wl.params, s.astype(np.float64), conditions=True)["abs_damp"]
    err = np.abs(a[1] - b[1][:L]) / terms
    print("damping gradients at v = %g, split against direct: %.1e" % (v0, err.max()))
    assert np.all(terms > 0) and err.max() <= 2.4e-7


@pytest.mark.parametrize("vmin", [17.0, 27.0, 90.0])
def test_microturbulence_gradient_far_out(gpu_lib, vmin):
    """dL/dxi from pixels where every line in reach has v >= vmin at every
    depth.  Its leading order in 1/v^2 cancels, so a power of the far zone's
    sum that H can do without shows here first.  The lines are weak and the
    seed positive, so the terms have one sign: each is good to 2e-6 (the powers
    left out 1e-6, float32 coefficients and products 1e-6), dL/dkappa and the
    sums' rounding (thousands of terms in float32) take the rest of 1e-5."""
    wl = W.tiny(seed=15, L=16, N=3001, D=24, S=4, xi=1.3, lam_lo=500.0, window_nm=4.0)
    lam = O.wavelengths_nm(wl.grid)
    wl.lines.lam0_nm[:] = np.random.default_rng(15).uniform(lam[1400], lam[1420], 16)
    wl.lines.loggf[:] = -6.0
    v = np.abs(_detunings(wl)).min(axis=(0, 2))
    i = np.arange(3001)
    s = np.where((v >= vmin) & (v < 2.0 * vmin + 20.0) & (np.abs(i - 1410) < 1300), 1.0, 0.0).astype(np.float32)
    assert s.sum() > 20
    g = gpu_vjp(gpu_lib, wl, s)
    ref = O.adjoint(wl, wl.params, s.astype(np.float64))
    err = abs(g[3][0] - ref["g_xi"]) / abs(ref["g_xi"])
    print("dL/dxi from v >= %g: relative error %.1e" % (vmin, err))
    assert err <= 1e-5
    np.testing.assert_allclose(g[0], ref["g_loggf"], rtol=1e-5)
