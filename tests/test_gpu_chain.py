"""Whole stages in one launch for the closed-form L^2 mixture and the 1D problem: every edge of the lane
layouts (modes per lane and chunk, components, likelihood terms, nodes per chunk, particles per wave
and workgroup) against the oracle's moves with the same random numbers.  Accept counts are equal;
states and potentials agree to the rounding of FP64 sums over at most 256 nodes and 128 modes (1e-10,
the bound of the other move tests).
"""
import sys

import numpy as np
import pytest
import torch

import inputs
from oracle import example1 as ex
from oracle.forward import phi as phi_pde
from oracle.moves import GM, gmpcn_moves
from oracle.problem import Problem as OProblem, active_modes

pytestmark = pytest.mark.gpu
DEV = "cuda"


def banner(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


def t(a, dtype=torch.float64):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device=DEV)


def check(p, N, K, kr, active, M, beta, tau, n_moves, phi_fn, spread):
    from paper_2503_16028_amd import smc
    xi0 = inputs.particles(N, K, 5, 0.9)
    phi0 = phi_fn(xi0)
    logw, mean, scale = inputs.mixture(M, kr, 6, spread=spread)
    xi, phi = t(xi0), t(phi0)
    acc = torch.empty(N, dtype=torch.int32, device=DEV)
    smc.smc_gmpcn_move(p, N, (t(logw), t(mean), t(scale)), beta, tau, n_moves, 9, 40, None, smc.SMC_FP64, xi, phi,
                       acc)
    assert smc.smc_status_flags(p) == 0
    rx, rphi, racc = gmpcn_moves(None, 0, xi0, phi0, GM(logw, mean, scale, active, K), beta, tau, n_moves, 9, 40,
                                 phi_fn=phi_fn)
    assert np.array_equal(acc.cpu().numpy(), racc)
    assert np.abs(xi.cpu().numpy() - rx).max() <= 1e-10 * np.abs(rx).max()
    assert np.abs(phi.cpu().numpy() / rphi - 1).max() <= 1e-10


# K, kr, likelihood terms, M, N, moves: a lane's modes end inside, at and past each chunk; every component
# and term block; one particle, a part of a workgroup, whole ones; a second batch of 16 moves
@pytest.mark.parametrize("K,kr,T,M,N,n_moves", [
    (1, 1, 1, 1, 1, 1), (9, 5, 3, 1, 17, 17), (32, 32, 4, 2, 33, 4), (33, 7, 5, 4, 3, 16), (64, 64, 16, 8, 16, 3),
    (65, 64, 4, 5, 15, 3), (64, 64, 2, 16, 50, 3), (127, 64, 16, 16, 5, 3), (128, 64, 4, 1, 21, 33),
    (64, 64, 4, 8, 4113, 1), (65, 7, 4, 5, 30, 8), (127, 9, 16, 16, 10, 16), (100, 6, 5, 8, 10, 17)])
def test_l2_mixture_stage(K, kr, T, M, N, n_moves):
    from paper_2503_16028_amd import smc
    banner("chain l2", K, kr, T, M, N, n_moves)
    prob = dict(ex.problem(K=max(K, 8)))                # the centres need eight modes
    prob.update(K=K, lam=prob["lam"][:K], sqrt_lam=prob["sqrt_lam"][:K],
                c=0.3 * np.random.default_rng(T).standard_normal((T, K)), sigma=0.5)
    p = smc.L2MixProblem(K, kr, prob["alpha"], prob["c"], prob["sigma"], N)
    check(p, N, K, kr, active_modes(prob["lam"], kr), M, 0.5, 0.7, n_moves, lambda x: ex.phi(prob, x), 0.4)


@pytest.mark.parametrize("n,kl,kr,M,N,n_moves", [
    (8, 5, 3, 1, 1, 1), (16, 9, 9, 2, 300, 2), (64, 64, 64, 8, 5, 17), (128, 33, 16, 16, 3, 3), (128, 12, 12, 4, 270, 2),
    (256, 64, 64, 1, 9, 3), (256, 20, 20, 8, 530, 1), (128, 33, 5, 16, 9, 5), (256, 64, 6, 3, 10, 6)])
def test_1d_stage(n, kl, kr, M, N, n_moves):
    from paper_2503_16028_amd import smc
    banner("chain 1d", n, kl, kr, M, N, n_moves)
    obs = sorted(set([1, n - 1] + [int(v) for v in np.linspace(1, n - 1, 12)]))
    d = dict(name="chain1d", dim=1, grids=[n], kl_per_axis=kl, kr=kr, obs_den=n, obs=[[o] for o in obs],
             y=list(0.1 * np.sin(np.arange(len(obs)) + 0.5)), sigma=0.2)
    op = OProblem(d)
    p = smc.Problem(d, N, grids=[n])
    check(p, N, kl, kr, op.active(), M, 0.4, 0.8, n_moves,
          lambda x: np.array([phi_pde(op, r, n) for r in np.atleast_2d(x)]) if np.ndim(x) > 1 else phi_pde(op, x, n), 0.4)
