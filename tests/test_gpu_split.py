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
