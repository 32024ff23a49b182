"""The near/far split of a line's window (far zone on the matrix cores, near
zone by direct evaluation) at the sizes where its tiles, k-steps, depth
groups and zone limits end, against the oracle.

Tolerance: every term of the opacity sum is positive, so the sum's relative
error is bounded by the terms': 1.4e-6 for the Voigt forms in use (the far
form 6e-8 + 6 float32 roundings of x/x0), 4e-7 for the float32 parameters and
at most 1e-6 for the float32 sums; 5e-6 covers them with a factor of 1.7.
"""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import synth as O

pytestmark = pytest.mark.gpu

KAPPA_RTOL = 5e-6


def _kappa(pz, wl, **kw):
    plan = pz.plan_for(wl, **kw)
    out = torch.empty((wl.atm.D, wl.grid.N), dtype=torch.float32, device="cuda")
    print("pz_line_opacity N=%d L=%d D=%d" % (wl.grid.N, wl.lines.L, wl.atm.D), flush=True)
    pz.pz_line_opacity(plan, pz.Atmos(wl.atm), pz.Params.from_host(wl.params), out)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


def _case(N, L, D, window_nm=0.3, lam=500.0, seed=5):
    wl = W.tiny(seed=seed, L=L, N=N, D=D, S=4, n_molecular=1, xi=1.3, lam_lo=lam, window_nm=window_nm)
    wl.params = W.random_params(np.random.default_rng(seed), L, 4, 1.3)
    return wl


@pytest.mark.parametrize("N,L,D,window", [
    (2, 1, 2, 0.3), (31, 3, 3, 0.3), (33, 5, 16, 0.3), (64, 63, 17, 0.3), (300, 65, 24, 0.3), (517, 129, 25, 0.3),
    (400, 40, 48, 0.3), (400, 40, 49, 0.3), (400, 31, 80, 0.3),
    (700, 200, 72, 0.012),        # windows narrower than the near zone: no far pixel
    (3001, 90, 20, 4.0),          # windows of 2,400 pixels: every far tier down to two powers
])
def test_split_sizes_vs_oracle(gpu_lib, N, L, D, window):
    wl = _case(N, L, D, window)
    ref = O.line_opacity(wl)
    np.testing.assert_allclose(_kappa(gpu_lib, wl), ref, rtol=KAPPA_RTOL, atol=1e-30)


@pytest.mark.parametrize("ddamp", [1.0, 2.0, 3.0])
def test_damped_lines_vs_oracle(gpu_lib, ddamp):
    """Damping ratios from below the small-damping limit to far above it: the
    zone limit moves outwards with the damping until a line has no far zone."""
    wl = _case(900, 70, 72, lam=1550.0)
    wl.params.ddamp = np.linspace(-1.0, ddamp, 70)
    np.testing.assert_allclose(_kappa(gpu_lib, wl), O.line_opacity(wl), rtol=KAPPA_RTOL)


def test_nonfinite_line_stays_in_its_window(gpu_lib):
    """A line whose strength overflows float32 spoils the pixels of its own
    window and no others (the matrix product would carry it to its tile)."""
    wl = _case(1200, 60, 72)
    wl.params.dgf[7] = 60.0
    got = _kappa(gpu_lib, wl)
    lam = O.wavelengths_nm(wl.grid)
    outside = np.abs(lam - wl.lines.lam0_nm[7]) > wl.window_nm
    assert outside.any() and not np.isfinite(got[:, ~outside]).all()
    keep = np.arange(60) != 7
    wl.lines, wl.params = wl.lines.take(keep), W.Params(wl.params.dgf[keep], wl.params.ddamp[keep], wl.params.dA, 1.3)
    np.testing.assert_allclose(got[:, outside], O.line_opacity(wl)[:, outside], rtol=KAPPA_RTOL, atol=1e-30)


@pytest.mark.parametrize("N,L,D,window,eta,fam", [
    (33, 1, 2, 0.3, 0.0, False), (300, 15, 16, 0.3, 0.0, True), (517, 17, 25, 0.3, 0.0, False),
    (400, 33, 49, 0.3, 1e-3, True), (400, 47, 80, 0.3, 0.0, True), (900, 65, 72, 0.3, 1e-3, False),
    (3001, 40, 20, 4.0, 0.0, False),
])
def test_split_gradients_vs_oracle(gpu_lib, N, L, D, window, eta, fam):
    """Line gradients at the ends of the 16-line, 16-pixel and 32-pixel steps of
    the gather, plain, with the centre test and per damping family (the rule of
    the other gradient tests: 1e-3 of a large entry, 1e-5 of the largest)."""
    from test_gpu_adjoint import grad_close_cond
    pz = gpu_lib
    wl = _case(N, L, D, window)
    wl.center_eta = eta
    if fam:
        rng = np.random.default_rng(3)
        wl.params.ddamp_family = rng.normal(0.0, 0.2, (3, L))
    s = np.random.default_rng(N).normal(size=N)
    plan = pz.plan_for(wl, flags=pz.PZ_FLAG_DAMPING_FAMILIES if fam else 0)
    e = lambda *n: torch.empty(n, device="cuda")  # noqa: E731
    g = [e(L), e(3, L) if fam else e(L), e(4), e(1)]
    seed = torch.as_tensor(s.astype(np.float32), device="cuda")
    print("synth_backward N=%d L=%d D=%d" % (N, L, D), flush=True)
    pz.synth_backward(plan, pz.Atmos(wl.atm), pz.Params.from_host(wl.params), seed, *g)
    got = [t.cpu().numpy().astype(np.float64) for t in g]
    ref = O.adjoint(wl, wl.params, s.astype(np.float32).astype(np.float64), conditions=True)
    grad_close_cond(got[0], ref["g_loggf"], ref["abs_loggf"], name="loggf")
    if fam:
        for f in range(3):
            grad_close_cond(got[1][f], ref["g_damp_family"][f], ref["abs_damp_family"][f], name="family %d" % f)
    else:
        grad_close_cond(got[1], ref["g_damp"], ref["abs_damp"], name="damp")
    grad_close_cond(got[2], ref["g_abund"], ref["abs_abund"], name="abund")
    grad_close_cond(got[3], ref["g_xi"], ref["abs_xi"], name="xi")
