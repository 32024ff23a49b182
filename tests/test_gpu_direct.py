"""The direct line sums and the direct gather, which plans with more than two
lines per pixel take on short grids: every LDS chunk count and tile width,
lines in the wide pass, tiles in halves against whole ones, the centre test and
the damping families, per star and in batches; against the oracle and bit for
bit against each other."""
import copy

import numpy as np
import pytest
import torch

import workloads as W
from oracle import synth as O
from test_gpu_adjoint import grad_close_cond

pytestmark = pytest.mark.gpu


def _dense(N, L, D, seed, window=0.05, lam=500.0, weak=0.0, eta=0.0):
    assert L > 2 * N
    wl = W.tiny(seed=seed, L=L, N=N, D=D, S=4, n_molecular=1, xi=1.2, lam_lo=lam, window_nm=window)
    wl.params = W.random_params(np.random.default_rng(seed), L, 4, 1.2)
    wl.lines.loggf = wl.lines.loggf - weak
    wl.center_eta = eta
    return wl


def _kappa(pz, wl, **kw):
    plan = pz.plan_for(wl, **kw)
    kap = torch.empty((wl.atm.D, wl.grid.N), dtype=torch.float32, device="cuda")
    print("pz_line_opacity N=%d L=%d D=%d eta=%g" % (wl.grid.N, wl.lines.L, wl.atm.D, wl.center_eta), kw, flush=True)
    pz.pz_line_opacity(plan, pz.Atmos(wl.atm), pz.Params.from_host(wl.params), kap)
    torch.cuda.synchronize()
    return kap.cpu().numpy()


def _close(wl, got):
    """The bounds of the other opacity tests; with the centre test a pixel at the
    edge of a span can flip (at most 3 eta kappa_c of one line)."""
    ref, kc = O.line_opacity(wl), O.continuum_opacity(wl)[None, :]
    err = np.abs(got.astype(np.float64) - ref)
    strict = err <= 2e-5 * ref + 2e-11 * kc + (1e-6 * kc if wl.center_eta else 0.0)
    assert np.mean(~strict) <= (1e-3 if wl.center_eta else 0.0)
    assert np.all(err[~strict] <= 6.0 * wl.center_eta * np.broadcast_to(kc, err.shape)[~strict])


@pytest.mark.parametrize("N,L", [(2, 5), (3, 8), (9, 20), (28, 59), (150, 310)])
@pytest.mark.parametrize("chunk", [1, 2, 3, 5, 7, 16])
@pytest.mark.parametrize("eta", [0.0, 1e-3])
def test_chunk_counts_and_tile_widths(gpu_lib, N, L, chunk, eta):
    """5 to 310 lines in chunks of 1 to 16: every chunk count from 1 up, odd and
    even (both ends of the double buffer), in tiles of 32, 64 and 128 pixels;
    the tile widths differ by the order of the lines alone."""
    wl = _dense(N, L, 72 if chunk > 2 else 17, 76, eta=eta)
    for tile in (32, 64, 128):
        _close(wl, _kappa(gpu_lib, wl, tile_px=tile, lines_per_chunk=chunk))


def _damping_jump(N, L, seed=77, eta=0.0):
    """Damping ratios from ~1 to ~3e4 over depth: every line is flagged for the wide pass."""
    wl = _dense(N, L, 24, seed, window=0.3, eta=eta)
    wl.atm = copy.deepcopy(wl.atm)
    wl.atm.npert[8:] *= 1e2
    wl.lines.log_gvdw[:] = -3.0
    wl.lines.log_gstark[:] = -12.0
    wl.lines.log_grad[:] = 5.0
    wl.lines.log_gvdw[::3] = -9.0                         # and some that are not
    return wl


@pytest.mark.parametrize("tile", [32, 64, 128])
@pytest.mark.parametrize("eta", [0.0, 1e-3])
def test_wide_pass(gpu_lib, tile, eta):
    wl = _damping_jump(120, 250, eta=eta)
    a = O.line_depth_params(wl.atm, wl.lines, wl.params.dgf, wl.params.ddamp, wl.params.dA, wl.params.xi_kms)["a"]
    assert np.sum((a.min(axis=1) < 8.0) & (a.max(axis=1) > 2.0e3)) > 50
    _close(wl, _kappa(gpu_lib, wl, tile_px=tile))


@pytest.mark.parametrize("D", [8, 24])
def test_halves_and_whole_tiles_bitwise(gpu_lib, D):
    """64-pixel tiles in halves (150 tiles) and whole (401): the first pixels of
    both grids see the same lines."""
    wl = _dense(25600, 6 * 25600, D, 78, lam=1500.0)
    short = copy.deepcopy(wl)
    short.grid = W.Grid(1500.0, wl.grid.R, 9600)
    keep = wl.lines.lam0_nm <= O.wavelengths_nm(short.grid)[-1] + 0.2
    short.lines = wl.lines.take(keep)
    short.params = W.Params(wl.params.dgf[keep], wl.params.ddamp[keep], wl.params.dA, 1.2)
    a, b = _kappa(gpu_lib, wl), _kappa(gpu_lib, short)
    np.testing.assert_array_equal(a[:, :9400], b[:, :9400])


@pytest.mark.parametrize("eta,fam", [(0.0, False), (0.0, True), (1e-3, False), (1e-3, True)])
@pytest.mark.parametrize("N,L,D", [(120, 260, 24), (97, 200, 72)])
def test_direct_gradients_vs_oracle(gpu_lib, N, L, D, eta, fam):
    pz = gpu_lib
    wl = _dense(N, L, D, 79, weak=3.0 if not eta else 1.0, eta=eta)
    if fam:
        wl.params.ddamp_family = np.random.default_rng(3).normal(0.0, 0.2, (3, L))
    s = np.random.default_rng(79).normal(size=N).astype(np.float32)
    plan = pz.plan_for(wl, flags=pz.PZ_FLAG_DAMPING_FAMILIES if fam else 0)
    e = lambda *n: torch.empty(n, device="cuda")  # noqa: E731
    g = [e(L), e(3, L) if fam else e(L), e(4), e(1)]
    print("synth_backward N=%d L=%d eta=%g fam=%d" % (N, L, eta, fam), flush=True)
    pz.synth_backward(plan, pz.Atmos(wl.atm), pz.Params.from_host(wl.params), torch.as_tensor(s, device="cuda"), *g)
    got = [t.cpu().numpy().astype(np.float64) for t in g]
    ref = O.adjoint(wl, wl.params, s.astype(np.float64), conditions=True)
    grad_close_cond(got[0], ref["g_loggf"], ref["abs_loggf"], name="loggf")
    for k in range(3 if fam else 1):
        r, a = (ref["g_damp_family"][k], ref["abs_damp_family"][k]) if fam else (ref["g_damp"], ref["abs_damp"])
        grad_close_cond(got[1][k] if fam else got[1], r, a, name="damp %d" % k)
    grad_close_cond(got[2], ref["g_abund"], ref["abs_abund"], name="abund")
    grad_close_cond(got[3], ref["g_xi"], ref["abs_xi"], name="xi")


@pytest.mark.parametrize("tile,chunk,eta", [(32, 3, 0.0), (64, 16, 0.0), (64, 1, 1e-3), (128, 5, 0.0), (128, 16, 1e-3)])
@pytest.mark.parametrize("skewed", [False, True])
def test_batch_of_direct_stars_bitwise(gpu_lib, tile, chunk, eta, skewed):
    """Dense stars of a batch (alike; or one with heavy tiles, which then go out
    in halves), one of them with lines of the wide pass, beside a star whose
    sums are split: each gets what its own calls give, bit for bit."""
    pz = gpu_lib
    wls = [_dense(700, 1500, 24, 80, eta=eta), _dense(433, 1000, 72, 81, eta=eta), _damping_jump(200, 450, eta=eta),
           W.tiny(seed=82, L=40, N=900, D=40, S=4, xi=1.0)]
    if skewed:
        wls.append(_dense(70, 2000, 24, 83, window=0.3, eta=eta))
    keep, stars = [], []
    e = lambda n: torch.full((n,), float("nan"), device="cuda")  # noqa: E731
    p = lambda t: t.data_ptr()  # noqa: E731
    for wl in wls:
        plan, atm, par = pz.plan_for(wl, tile_px=tile, lines_per_chunk=chunk), pz.Atmos(wl.atm), pz.Params.from_host(wl.params)
        out = [e(plan.N), e(plan.N), e(plan.L), e(plan.L), e(plan.S), e(1)]
        seed = torch.as_tensor(np.random.default_rng(plan.N).normal(size=plan.N).astype(np.float32), device="cuda")
        keep.append((plan, atm, par, out, seed))
        stars.append(pz.pz_star(plan.handle, atm.c, par.c, p(out[0]), p(out[1]), p(seed), None, 0.0, None, *map(p, out[2:])))
    batch = pz.Batch(stars)
    print("synth_batch of %d stars, tile %d" % (len(wls), tile), flush=True)
    pz.synth_batch(batch, pz.PZ_MODE_FWD_BWD)
    torch.cuda.synchronize()
    for plan, atm, par, out, seed in keep:
        one = [e(t.numel()) for t in out]
        pz.synth_forward(plan, atm, par, one[0], one[1])
        pz.synth_backward(plan, atm, par, seed, *one[2:])
        torch.cuda.synchronize()
        for x, y in zip(out, one):
            np.testing.assert_array_equal(x.cpu().numpy(), y.cpu().numpy())


def test_autotune_of_split_and_direct_plans(gpu_lib):
    """A plan that splits its sums does not depend on the pair: the tuner returns
    the same one each time instead of the fastest of six equal ones."""
    pz = gpu_lib
    for wl, want in ((W.tiny(seed=9, L=300, N=3000, D=24), {(32, 16)}),
                     (_dense(300, 700, 24, 84), {(t, c) for t in (32, 64, 128) for c in (8, 16)})):
        for _ in range(4):
            tile, chunk, ms = pz.pz_autotune(wl.grid, wl.lines, wl.atm.S, wl.atm.D, pz.Atmos(wl.atm),
                                             pz.Params.from_host(wl.params), reps=2)
            assert (tile, chunk) in want and ms > 0
