"""The gather of the split line sums (near zone by direct evaluation, far zone
as a matrix product) against the direct gather and the oracle, at detunings
where the forms of the Voigt derivatives in use differ most."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import synth as O
from test_gpu_adjoint import gpu_vjp, grad_close_cond

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
    """Damping gradients of weak lines from one pixel, near |v| = v0 of a line:
    for the lines that have the pixel in their near zone the split gather and
    the direct one evaluate the same form of a dH/da there and add its eight
    depths in the same order.  The lines are too weak for the opacity's
    rounding to show in dL/dkappa by more than one rounding: 2.4e-7 of the sum
    of the terms' magnitudes, two units in the last place."""
    L = 90                                                # 34 windows over a pixel: a plan that splits the gather
    wl = W.tiny(seed=14, L=L, N=800, D=8, S=4, xi=2.0, lam_lo=500.0)
    wl.lines.loggf[:] = -10.0
    v = np.abs(_detunings(wl))
    k = int(np.argsort(wl.lines.lam0_nm)[L // 2])
    i = int(np.argmin(np.abs(v[k].mean(axis=1) - v0)))
    s = np.zeros(wl.grid.N, np.float32)
    s[i] = 1.0
    near = v[:, i].max(axis=1) < 5.4
    assert near[k] and np.all(O.line_opacity(wl) < 1e-3 * O.continuum_opacity(wl)[None, :])
    a, b = gpu_vjp(gpu_lib, wl, s), gpu_vjp(gpu_lib, _dense(wl), s)
    terms = O.adjoint(wl, wl.params, s.astype(np.float64), conditions=True)["abs_damp"]
    err = np.abs(a[1] - b[1][:L])[near] / terms[near]
    print("damping gradients at v = %g, split against direct: %.1e (%d lines)" % (v0, err.max(), near.sum()))
    assert err.max() <= 2.4e-7


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


def _check_gradients(pz, wl, s, fam):
    L = wl.lines.L
    plan = pz.plan_for(wl, flags=pz.PZ_FLAG_DAMPING_FAMILIES if fam else 0)
    e = lambda *n: torch.empty(n, device="cuda")  # noqa: E731
    g = [e(L), e(3, L) if fam else e(L), e(wl.atm.S), e(1)]
    print("synth_backward N=%d L=%d D=%d" % (wl.grid.N, L, wl.atm.D), flush=True)
    pz.synth_backward(plan, pz.Atmos(wl.atm), pz.Params.from_host(wl.params), torch.as_tensor(s, device="cuda"), *g)
    got = [t.cpu().numpy().astype(np.float64) for t in g]
    ref = O.adjoint(wl, wl.params, s.astype(np.float64), conditions=True)
    grad_close_cond(got[0], ref["g_loggf"], ref["abs_loggf"], name="loggf")
    if fam:
        for f in range(3):
            grad_close_cond(got[1][f], ref["g_damp_family"][f], ref["abs_damp_family"][f], name="family %d" % f)
    else:
        grad_close_cond(got[1], ref["g_damp"], ref["abs_damp"], name="damp")
    grad_close_cond(got[2], ref["g_abund"], ref["abs_abund"], name="abund")
    grad_close_cond(got[3], ref["g_xi"], ref["abs_xi"], name="xi")


@pytest.mark.parametrize("N,L,D,eta,fam", [
    (256, 31, 2, 0.0, False), (257, 32, 16, 0.0, True), (271, 33, 17, 0.0, False), (272, 47, 33, 1e-30, True),
    (273, 48, 48, 0.0, True), (400, 49, 49, 1e-30, False), (517, 65, 72, 0.0, False), (517, 80, 80, 0.0, True),
    (900, 129, 72, 0.0, False),
])
def test_split_gather_sizes_vs_oracle(gpu_lib, N, L, D, eta, fam):
    """Gradients where the windows overlap enough for the gather to be split: at
    the ends of its 16-line, 16-pixel and 16-depth steps, plain, per damping
    family and with a centre test that keeps everything (the rule of the other
    gradient tests: 1e-3 of a large entry, 1e-5 of the largest)."""
    wl = W.tiny(seed=N + L, L=L, N=N, D=D, S=4, n_molecular=1, xi=1.3, lam_lo=500.0)
    wl.params = W.random_params(np.random.default_rng(L), L, 4, 1.3)
    wl.center_eta = eta
    if fam:
        wl.params.ddamp_family = np.random.default_rng(3).normal(0.0, 0.2, (3, L))
    _check_gradients(gpu_lib, wl, np.random.default_rng(N).normal(size=N).astype(np.float32), fam)


def test_lines_in_distant_clusters(gpu_lib):
    """Windows that overlap within clusters and leave thousands of pixels
    between them: sixteen neighbouring lines of a far step can belong to two
    clusters, and the walk passes over the pixels between.  One line beyond
    the last pixel, out of reach."""
    N, L = 20011, 1500
    wl = W.tiny(seed=44, L=L, N=N, D=12, S=4, n_molecular=1, xi=1.3, lam_lo=500.0)
    lam = O.wavelengths_nm(wl.grid)
    rng = np.random.default_rng(44)
    c = np.concatenate([rng.uniform(900, 1300, 713), rng.uniform(9000, 9200, 778), rng.uniform(19900, 20011, 8)])
    wl.lines.lam0_nm[:-1] = 500.0 * (1.0 + 1.0 / wl.grid.R) ** c
    wl.lines.lam0_nm[-1] = lam[-1] + 0.7
    wl.params = W.random_params(rng, L, 4, 1.3)
    _check_gradients(gpu_lib, wl, rng.normal(size=N).astype(np.float32), False)


@pytest.mark.parametrize("N,L,window", [(3000, 15, 0.3), (20000, 40, 0.3), (2000, 900, 0.03)])
def test_plans_that_split_the_opacity_only(gpu_lib, N, L, window):
    """Sparse lines and narrow windows keep the direct gather."""
    wl = W.tiny(seed=45, L=L, N=N, D=24, S=4, n_molecular=1, xi=1.3, lam_lo=500.0, window_nm=window)
    wl.params = W.random_params(np.random.default_rng(45), L, 4, 1.3)
    _check_gradients(gpu_lib, wl, np.random.default_rng(45).normal(size=N).astype(np.float32), False)
