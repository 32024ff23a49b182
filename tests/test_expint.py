"""E_3 as a power series up to x = 1 and a polynomial per octave beyond
(expint_consts.h): the constants against scipy's expn, and the E2 flux on the
GPU with optical depths at the edges of the octaves."""
import math
import os
import re

import numpy as np
import pytest
import torch
from scipy.special import expn

from oracle import synth as O

HEADER = os.path.join(os.path.dirname(__file__), "..", "paper_2607_24141_amd", "csrc", "expint_consts.h")


def _constants():
    with open(HEADER) as f:
        text = f.read().replace("\\\n", "")
    get = lambda n: [float(v) for v in re.search(r"#define %s (.*)" % n, text).group(1).split(",")]  # noqa: E731
    rows = int(get("PZ_E3_OCTAVES")[0])
    return get("PZ_E3_PSI")[0], get("PZ_E3_SERIES"), np.array(get("PZ_E3_TABLE")).reshape(rows, -1)


def _e3(x, psi, series, table):
    if x <= 1.0:
        p = 0.0
        for c in series[::-1]:
            p = p * x + c
        return 0.5 - x + x * x * (0.5 * (psi - math.log(x)) + x * p)
    o = min(math.frexp(x)[1] - 1, len(table) - 1)
    hi = 0.5 ** o
    lo = 0.0 if o == len(table) - 1 else hi / 2
    t, p = (1.0 / x - lo) * (2.0 / (hi - lo)) - 1.0, 0.0
    for c in table[o][::-1]:
        p = p * t + c
    return math.exp(-x) / x * p


@pytest.mark.parametrize("lo,hi", [(1e-12, 1e-3), (1e-3, 1.0), (1.0, 2.0), (2.0, 4.0), (4.0, 8.0), (8.0, 16.0), (16.0, 700.0)])
def test_constants_vs_expn(lo, hi):
    # the series' terms sum to 14 times E_3 at x = 1: 14 x 2 roundings of 1.1e-16, and scipy's own
    x = np.concatenate([np.geomspace(lo, hi, 4001), [np.nextafter(lo, 1e3), np.nextafter(hi, 0.0)]])
    c = _constants()
    np.testing.assert_allclose([_e3(v, *c) for v in x], expn(3, x), rtol=1e-14)


@pytest.mark.gpu
@pytest.mark.parametrize("edge", [1.0, 2.0, 4.0, 8.0, 16.0, 700.0])
def test_e2_flux_at_octave_edges(gpu_lib, edge):
    """Knots at an edge, one float32 step to either side of it, and far from it."""
    e = np.float32(edge)
    tau = np.sort(np.float32([1e-3, 0.3 * e, np.nextafter(e, np.float32(0)), e, np.nextafter(e, np.float32(1e4)),
                              3.0 * e, 1e3 * e]))[:, None] * np.ones((1, 3), np.float32)
    S = (np.float32([1.0, 2.0, 0.5])[None, :] * (1.0 + tau) ** np.float32([0.25, 0.5, 1.0])[None, :]).astype(np.float32)
    F = torch.empty(3, dtype=torch.float32, device="cuda")
    print("pz_debug_formal_solve E2, knots at", edge, flush=True)
    gpu_lib.pz_debug_formal_solve(torch.as_tensor(S, device="cuda"), torch.as_tensor(tau, device="cuda"), F, quadrature=1)
    torch.cuda.synchronize()
    # one float32 rounding of a float64 sum
    np.testing.assert_allclose(F.cpu().numpy(), O.flux_e2(S.astype(float), tau.astype(float)), rtol=2e-7)
