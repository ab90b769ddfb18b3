"""Every tile of the on-chip solver (GPU): a call that wants the observations alone takes no longer than one that
keeps the whole solution as well, and gives the same observations to the solver's tolerance.  On chip the
solution adds to a solve an iterate read and written in each of three sweeps, beside the transforms of nine
iterations: less than four tenths."""
import json
import sys

import numpy as np
import pytest
import torch

from conftest import golden

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n,rows,prec", [(32, 4, 1), (32, 8, 1), (64, 4, 1), (64, 8, 1), (64, 16, 1), (128, 16, 1),
                                         (128, 32, 1), (256, 0, 1), (64, 0, 0), (128, 0, 0), (256, 0, 0)])
def test_observations_cost_no_more_than_the_state(n, rows, prec):
    from paper_2503_16028_amd import smc
    print("[case] observations and state", n, rows, prec, flush=True)
    sys.stdout.flush()
    N = 2048 if n < 256 else 256
    d = json.load(open(golden("problem_t2.json")))
    d.update(grids=[n], kl_per_axis=32)
    p = smc.Problem(d, N)
    if rows:
        smc.smc_set_tile(p, 0, rows)
    xi = torch.randn(N, p.K, generator=torch.Generator(device=DEV).manual_seed(n), dtype=torch.float64, device=DEV)
    G, K = (torch.empty(N, p.n_obs, dtype=torch.float64, device=DEV) for _ in range(2))
    w = torch.empty(N, n * n, dtype=torch.float64, device=DEV)

    def best(f):
        out = np.inf
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        for _ in range(5):
            a.record()
            f()
            f()
            b.record()
            torch.cuda.synchronize()
            out = min(out, a.elapsed_time(b) / 2)
        return out

    obs = best(lambda: smc.smc_forward_batch(p, N, xi, None, prec, G))
    state = best(lambda: smc.smc_forward_state(p, N, xi, prec, K, w))
    print("   observations %.3f ms, state %.3f ms" % (obs, state), flush=True)
    assert smc.smc_status_flags(p) == 0
    assert ((G - K).abs().amax(1) <= 2e-9 * K.abs().amax(1)).all()   # each to 1e-9 of the exact ones
    assert obs <= 1.1 * state
    if prec == 1 and n < 256:
        assert state <= 1.4 * obs


@pytest.mark.parametrize("n,prec", [(256, 1), (256, 0), (128, 0)])
def test_gradient_costs_little_more_than_the_state(n, prec):
    """From kept states a gradient is one adjoint solve, to the forward solve's tolerance and with its passes, and a
    contraction that reads three fields where the solve moves fifty: less than a fifth more."""
    from paper_2503_16028_amd import smc
    print("[case] gradient and state", n, prec, flush=True)
    N = 300
    d = json.load(open(golden("problem_t2.json")))
    d.update(grids=[n], kl_per_axis=32, obs_den=16, obs=[[i, j] for i in range(3, 13, 2) for j in range(3, 13, 2)],
             y=[0.05] * 25)
    p = smc.Problem(d, N)
    xi = torch.randn(N, p.K, generator=torch.Generator(device=DEV).manual_seed(n), dtype=torch.float64, device=DEV)
    G = torch.empty(N, p.n_obs, dtype=torch.float64, device=DEV)
    w = torch.empty(N, n * n, dtype=torch.float64, device=DEV)
    phi, grad = torch.empty(N, dtype=torch.float64, device=DEV), torch.empty_like(xi)

    def best(f):
        out = np.inf
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        for _ in range(5):
            a.record()
            f()
            b.record()
            torch.cuda.synchronize()
            out = min(out, a.elapsed_time(b))
        return out

    state = best(lambda: smc.smc_forward_state(p, N, xi, prec, G, w))
    gradient = best(lambda: smc.smc_value_and_grad(p, N, xi, prec, w, phi, grad))
    print("   state %.3f ms, gradient %.3f ms" % (state, gradient), flush=True)
    assert smc.smc_status_flags(p) == 0 and torch.isfinite(grad).all()
    assert gradient <= 1.2 * state
