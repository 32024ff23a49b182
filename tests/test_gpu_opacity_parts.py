"""Direct line sums with a tile in two workgroups (few tiles) and in one (many),
against the oracle, at depth counts with and without a tail of depths."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import synth as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,D,N,L", [
    (64, 2, 130, 300), (64, 8, 130, 300), (64, 17, 200, 500), (64, 72, 200, 450), (64, 80, 65, 200),
    (128, 17, 300, 700), (128, 72, 129, 300), (32, 17, 130, 300),
])
@pytest.mark.parametrize("eta", [0.0, 1e-3])
def test_direct_sums_vs_oracle(gpu_lib, tile, D, N, L, eta):
    wl = W.tiny(seed=8, L=L, N=N, D=D, S=4, n_molecular=1, xi=1.3, lam_lo=500.0, window_nm=0.05)
    wl.params = W.random_params(np.random.default_rng(8), L, 4, 1.3)
    wl.center_eta = eta
    plan = gpu_lib.plan_for(wl, tile_px=tile, center_eta=eta)
    F = torch.empty(plan.N, dtype=torch.float32, device="cuda")
    Fc = torch.empty_like(F)
    print("synth_forward tile=%d D=%d N=%d L=%d eta=%g" % (tile, D, N, L, eta), flush=True)
    gpu_lib.synth_forward(plan, gpu_lib.Atmos(wl.atm), gpu_lib.Params.from_host(wl.params), F, Fc)
    torch.cuda.synchronize()
    ref = O.synthesize(wl)
    # the path's flux tolerance against the oracle
    np.testing.assert_allclose(F.cpu().numpy() / Fc.cpu().numpy(), ref[0] / ref[1], rtol=1e-4)
