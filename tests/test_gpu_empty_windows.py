"""Windows narrower than the pixel spacing: most lines lie between two pixels
with none within W and add nothing, the others reach one pixel.  Opacity and
line gradients against the oracle, plain and with the centre test, on sparse
grids (split line sums) and on dense ones (direct)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import synth as O
from test_gpu_adjoint import gpu_vjp, grad_close_cond

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,R,window", [(400, 60, 3.0e5, 5.0e-4), (397, 300, 1.0e4, 0.02), (203, 700, 3.0e5, 3.0e-4)])
@pytest.mark.parametrize("eta", [0.0, 1e-3])
def test_windows_below_a_pixel(gpu_lib, N, L, R, window, eta):
    wl = W.tiny(seed=19, L=L, N=N, D=24, S=4, n_molecular=1, xi=1.3, lam_lo=500.0, window_nm=window)
    wl.grid = W.Grid(500.0, R, N)
    lam = O.wavelengths_nm(wl.grid)
    wl.lines.lam0_nm = np.random.default_rng(19).uniform(lam[0] - 3.0 * window, lam[-1] + 3.0 * window, L)
    wl.params = W.random_params(np.random.default_rng(19), L, 4, 1.3)
    wl.center_eta = eta
    p_idx, l_idx = O.window_pairs(wl.grid, wl.lines, window, np.arange(N))
    assert 0 < len(set(l_idx)) < 0.9 * L                  # some lines reach a pixel, others none
    plan = gpu_lib.plan_for(wl)
    kap = torch.empty((24, N), dtype=torch.float32, device="cuda")
    print("pz_line_opacity N=%d L=%d window=%g eta=%g" % (N, L, window, eta), flush=True)
    gpu_lib.pz_line_opacity(plan, gpu_lib.Atmos(wl.atm), gpu_lib.Params.from_host(wl.params), kap)
    # the tolerance of the split sums' tests
    np.testing.assert_allclose(kap.cpu().numpy().astype(np.float64), O.line_opacity(wl), rtol=5e-6, atol=1e-30)
    s = np.random.default_rng(N).normal(size=N).astype(np.float32)
    g = gpu_vjp(gpu_lib, wl, s)
    ref = O.adjoint(wl, wl.params, s.astype(np.float64), conditions=True)
    grad_close_cond(g[0], ref["g_loggf"], ref["abs_loggf"], name="loggf")
    grad_close_cond(g[1], ref["g_damp"], ref["abs_damp"], name="damp")
    grad_close_cond(g[2], ref["g_abund"], ref["abs_abund"], name="abund")
