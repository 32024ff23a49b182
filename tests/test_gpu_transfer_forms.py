"""The transfer's two forms, a row of sixteen lanes per pixel and one thread per
pixel, at depth counts that fill two to five depths per lane and at grids on
both sides of the rule between the forms: fluxes and dL/dkappa against the
oracle, and the two forms of the Gauss-3 flux against each other."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import scatter as SC
from oracle import synth as O
from test_gpu_forward import _flux_close, _run_forward

pytestmark = pytest.mark.gpu


def _wl(N, D, quad="gauss3", L=60, seed=23):
    wl = W.tiny(seed=seed, L=L, N=N, D=D, S=4, n_molecular=1, xi=1.2, lam_lo=600.0, window_nm=0.2)
    wl.params = W.random_params(np.random.default_rng(seed), L, 4, 1.2)
    wl.lines.lam0_nm = np.sort(np.random.default_rng(seed).uniform(600.0, 602.0, L))     # the first 1,000 pixels
    wl.quadrature = quad
    wl.atm.lam_ref_nm = 600.0                             # the same physics at every grid length
    return wl


# rows: two to five depths per lane, full and ragged; columns: from the grid lengths named
FORMS = [("gauss3", 400, 20), ("gauss3", 400, 33), ("gauss3", 400, 48), ("gauss3", 400, 57), ("gauss3", 400, 65),
         ("gauss3", 60000, 2), ("gauss3", 60001, 8), ("gauss3", 120011, 33), ("gauss3", 361193, 72),
         ("e2", 400, 2), ("e2", 400, 20), ("e2", 400, 33), ("e2", 400, 48), ("e2", 400, 64), ("e2", 400, 80),
         ("e2", 20003, 2), ("e2", 40001, 16), ("e2", 100003, 49)]


@pytest.mark.parametrize("quad,N,D", FORMS)
def test_transfer_forms_vs_oracle(gpu_lib, quad, N, D):
    pz = gpu_lib
    wl = _wl(N, D, quad)
    plan = pz.plan_for(wl)
    F, Fc = _run_forward(pz, wl, plan)
    pix = np.unique(np.concatenate([np.arange(0, 400, 9), np.linspace(0, N - 1, 40).astype(int)]))
    kl = O.line_opacity(wl, pix=pix)
    _flux_close(F[pix], Fc[pix], *O.synthesize(wl, pix=pix))
    s = np.random.default_rng(N).normal(size=N).astype(np.float32)
    g = torch.empty((D, N), device="cuda")
    print("pz_debug_opacity_adjoint", quad, N, D, flush=True)
    pz.pz_debug_opacity_adjoint(plan, pz.Atmos(wl.atm), pz.Params.from_host(wl.params), torch.as_tensor(s, device="cuda"), g)
    ref = O.opacity_adjoint(wl, kl, s[pix].astype(np.float64), pix)
    err = np.abs(g.cpu().numpy()[:, pix] - ref) / np.max(np.abs(ref), axis=0, keepdims=True)
    print("%s N %d D %d: dL/dkappa within %.1e" % (quad, N, D, err.max()))
    assert err.max() <= 2e-5                              # the tolerance of the reverse scan's other tests


@pytest.mark.parametrize("D,n_rows,n_columns", [(8, 20001, 60000), (33, 20001, 120000), (4, 4001, 60000)])
def test_gauss3_flux_forms_bitwise(gpu_lib, D, n_rows, n_columns):
    """The same pixels on a short grid (rows) and a long one (columns): the
    Gauss-3 flux walks the depths in the same order either way."""
    a = _run_forward(gpu_lib, _wl(n_rows, D))
    b = _run_forward(gpu_lib, _wl(n_columns, D))
    n = 3000                                              # all line windows, and continuum
    for x, y in zip(a, b):
        np.testing.assert_array_equal(np.asarray(x)[:n], np.asarray(y)[:n])


def test_batch_of_both_forms_bitwise(gpu_lib):
    """Stars of a batch whose transfer goes by rows and by columns get what
    their own calls give, bit for bit."""
    pz = gpu_lib
    wls = [_wl(N, D, quad, seed=30 + k) for k, (quad, N, D) in
           enumerate([("gauss3", 500, 20), ("gauss3", 60001, 8), ("e2", 500, 33), ("e2", 40001, 16), ("gauss3", 131100, 4)])]
    keep, stars = [], []
    e = lambda n: torch.full((n,), float("nan"), device="cuda")  # noqa: E731
    p = lambda t: t.data_ptr()  # noqa: E731
    for wl in wls:
        plan, atm, par = pz.plan_for(wl), pz.Atmos(wl.atm), pz.Params.from_host(wl.params)
        out = [e(plan.N), e(plan.N), e(plan.L), e(plan.L), e(plan.S), e(1)]
        seed = torch.as_tensor(np.random.default_rng(plan.N).normal(size=plan.N).astype(np.float32), device="cuda")
        keep.append((plan, atm, par, out, seed))
        stars.append(pz.pz_star(plan.handle, atm.c, par.c, p(out[0]), p(out[1]), p(seed), None, 0.0, None, *map(p, out[2:])))
    batch = pz.Batch(stars)
    print("synth_batch of five stars", flush=True)
    pz.synth_batch(batch, pz.PZ_MODE_FWD_BWD)
    torch.cuda.synchronize()
    for plan, atm, par, out, seed in keep:
        one = [e(t.numel()) for t in out]
        pz.synth_forward(plan, atm, par, one[0], one[1])
        pz.synth_backward(plan, atm, par, seed, *one[2:])
        torch.cuda.synchronize()
        for x, y in zip(out, one):
            np.testing.assert_array_equal(x.cpu().numpy(), y.cpu().numpy())


@pytest.mark.parametrize("D", [33, 48, 57, 64])
def test_scattering_with_three_and_four_depths_per_lane(gpu_lib, D):
    """Fluxes to 1e-5 and dL/dkappa to 2e-5 of each pixel's largest, the
    tolerances of the other scattering tests."""
    pz = gpu_lib
    wl = _wl(300, D, L=20)
    wl.atm.sigma_c = 1.5 * (1.0 + 0.5 * np.sin(0.7 * np.arange(D)))
    plan = pz.plan_for(wl)
    F, Fc = _run_forward(pz, wl, plan)
    Fo, Fco = SC.synthesize(wl)
    assert max(np.max(np.abs(F / Fo - 1)), np.max(np.abs(Fc / Fco - 1))) <= 1e-5
    s = np.random.default_rng(D).normal(size=300).astype(np.float32)
    g = torch.empty((D, 300), device="cuda")
    print("scatter adjoint D=%d" % D, flush=True)
    pz.pz_debug_opacity_adjoint(plan, pz.Atmos(wl.atm), pz.Params.from_host(wl.params), torch.as_tensor(s, device="cuda"), g)
    ref = SC.opacity_adjoint(wl, O.line_opacity(wl), s.astype(np.float64))
    err = np.abs(g.cpu().numpy() - ref) / np.max(np.abs(ref), axis=0, keepdims=True)
    assert err.max() <= 2e-5
