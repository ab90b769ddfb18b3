"""Which route a stage of the closed-form L^2 mixture or the 1D problem takes for a large cloud (GPU): in one
launch, or by steps where its tables cost more than its moves save.  Both give the oracle's moves (accept counts
equal, 1e-10 as in the other move tests), on either side of each line; and a single move of a large cloud on a
coarse grid costs no more than its proposal and potential by themselves, with a third for the decision."""
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


def check(p, N, K, kr, active, M, n_moves, phi_fn):
    """All N rows on the device; 200 of them, the ends among them, by the oracle."""
    from paper_2503_16028_amd import smc
    xi0 = inputs.particles(N, K, 5, 0.9)
    ids = np.unique(np.concatenate([[0, 1, N - 2, N - 1], np.random.default_rng(N).choice(N, 196, replace=False)]))
    logw, mean, scale = inputs.mixture(M, kr, 6, spread=0.4)
    xi, phi = t(xi0), torch.empty(N, dtype=torch.float64, device=DEV)
    acc = torch.empty(N, dtype=torch.int32, device=DEV)
    smc.smc_phi_batch(p, N, xi, None, smc.SMC_FP64, phi)
    phi0 = np.array([phi_fn(x) for x in xi0[ids]])
    assert np.abs(phi.cpu().numpy()[ids] / phi0 - 1).max() <= 1e-10
    smc.smc_gmpcn_move(p, N, (t(logw), t(mean), t(scale)), 0.5, 0.7, n_moves, 9, 40, None, smc.SMC_FP64, xi, phi, acc)
    assert smc.smc_status_flags(p) == 0
    rx, rphi, racc = gmpcn_moves(None, 0, xi0[ids], phi0, GM(logw, mean, scale, active, K), 0.5, 0.7, n_moves, 9, 40,
                                 phi_fn=phi_fn, ids=ids)
    assert np.array_equal(acc.cpu().numpy()[ids], racc) and racc.sum() > 0
    assert np.abs(xi.cpu().numpy()[ids] - rx).max() <= 1e-10 * np.abs(rx).max()
    assert np.abs(phi.cpu().numpy()[ids] / rphi - 1).max() <= 1e-10


@pytest.mark.parametrize("K,T,M,N,n_moves", [(9, 1, 16, 32769, 1), (9, 1, 16, 32768, 1), (50, 3, 8, 32770, 1),
                                             (9, 1, 16, 32769, 3)])
def test_l2_mixture_routes(K, T, M, N, n_moves):
    from paper_2503_16028_amd import smc
    banner("route l2", K, T, M, N, n_moves)
    prob = dict(ex.problem(K=max(K, 8)))
    prob.update(K=K, lam=prob["lam"][:K], sqrt_lam=prob["sqrt_lam"][:K],
                c=0.3 * np.random.default_rng(T).standard_normal((T, K)), sigma=0.5)
    p = smc.L2MixProblem(K, K, prob["alpha"], prob["c"], prob["sigma"], N)
    check(p, N, K, K, active_modes(prob["lam"], K), M, n_moves, lambda x: ex.phi(prob, x))


@pytest.mark.parametrize("n,K,M,N,n_moves", [(8, 5, 3, 8193, 1), (8, 5, 3, 8192, 1), (16, 9, 3, 8193, 1),
                                             (8, 5, 16, 8200, 2)])
def test_1d_routes(n, K, M, N, n_moves):
    from paper_2503_16028_amd import smc
    banner("route 1d", n, K, M, N, n_moves)
    obs = sorted(set([1, n - 1] + [int(v) for v in np.linspace(1, n - 1, 6)]))
    d = dict(name="route1d", dim=1, grids=[n], kl_per_axis=K, kr=K, obs_den=n, obs=[[o] for o in obs],
             y=list(0.1 * np.sin(np.arange(len(obs)) + 0.5)), sigma=0.2)
    op = OProblem(d)
    p = smc.Problem(d, N, grids=[n])
    check(p, N, K, K, op.active(), M, n_moves, lambda x: phi_pde(op, x, n))


@pytest.mark.parametrize("kind,n,K,M", [("1d", 8, 8, 16), ("1d", 16, 16, 16), ("1d", 32, 4, 16), ("l2", 0, 16, 16)])
def test_one_move_of_a_large_cloud(kind, n, K, M):
    from paper_2503_16028_amd import smc
    banner("one move", kind, n, K, M)
    N = 262144
    if kind == "1d":
        d = dict(dim=1, grids=[n], kl_per_axis=K, kr=K, obs=[[i] for i in range(1, 8)], obs_den=8, y=[0.0] * 7,
                 sigma=0.2)
        p = smc.Problem(d, N)
    else:
        p = smc.L2MixProblem(K, K, 0.01, np.full((1, K), 0.1), 0.3, N)
    xi = torch.randn(N, K, generator=torch.Generator(device=DEV).manual_seed(1), dtype=torch.float64, device=DEV)
    v, (phi, logr) = torch.empty_like(xi), (torch.empty(N, dtype=torch.float64, device=DEV) for _ in range(2))
    acc = torch.empty(N, dtype=torch.int32, device=DEV)
    gm = tuple(t(a) for a in inputs.mixture(M, K, 6, spread=0.4))
    smc.smc_phi_batch(p, N, xi, None, smc.SMC_FP64, phi)

    def best(f):
        out = np.inf
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        for _ in range(6):
            a.record()
            f()
            f()
            b.record()
            torch.cuda.synchronize()
            out = min(out, a.elapsed_time(b) / 2)
        return out

    def parts():
        smc.smc_gmpcn_propose(p, N, gm, 0.3, 3, 1000, xi, v, logr)
        smc.smc_phi_batch(p, N, v, None, smc.SMC_FP64, logr)

    steps = best(parts)
    move = best(lambda: smc.smc_gmpcn_move(p, N, gm, 0.3, 0.3, 1, 3, 1000, None, smc.SMC_FP64, xi, phi, acc))
    print("   parts %.3f ms, move %.3f ms" % (steps, move), flush=True)
    assert move <= 4.0 / 3.0 * steps
