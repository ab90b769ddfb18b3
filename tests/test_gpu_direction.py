"""The transform of the solver with its vectors in memory, on a residual that has grown since its scale was
taken (GPU): between two iterations the residual is staged in FP16 at the scale of its norm before the
update, and one that has outgrown the scale must be staged anew.

Tolerance: that of the preconditioner's own test, 4e-3 of the largest value, from FP16 operands (2^-11 each) in
four products; the scale is a power of two, so at unchanged precision it adds nothing.
"""
import json
import sys

import numpy as np
import pytest
import torch

import inputs
from conftest import golden

pytestmark = pytest.mark.gpu
DEV = "cuda"


def reference(r, n):
    a = np.arange(1, n)
    S = np.sqrt(2.0 / n) * np.sin(np.pi * np.outer(a, a) / n)
    lam = np.sin(np.pi * a / (2 * n)) ** 2
    return S @ ((S @ r[:n - 1, :n - 1] @ S) / (lam[:, None] + lam[None, :])) @ S


@pytest.mark.parametrize("n", [128, 256])
@pytest.mark.parametrize("growth", [1.0, 5.0, 45.0, 300.0, 5000.0, 1e7])
def test_residual_that_outgrew_its_scale(n, growth):
    from paper_2503_16028_amd import smc
    print("[case] staged transform", n, growth, flush=True)
    sys.stdout.flush()
    d = json.load(open(golden("problem_t2.json")))
    d.update(grids=[n])
    p = smc.Problem(d, 3)
    s = np.sin(np.pi * np.arange(1, n + 1) / n)
    r = np.zeros((3, n, n), dtype=np.float32)
    r[0] = np.outer(s, s)                                        # the lowest mode: the largest quotient
    r[1] = np.outer(s, np.sin(3 * np.pi * np.arange(1, n + 1) / n))
    r[2] = inputs.particles(n, n, 5)
    r[:, n - 1, :] = 0.0
    r[:, :, n - 1] = 0.0
    r /= np.sqrt((r.astype(np.float64) ** 2).sum((1, 2)))[:, None, None]
    z = torch.empty(3, n, n, dtype=torch.float32, device=DEV)
    smc.smc_precond_apply_staged(p, 0, 3, torch.tensor(r, device=DEV), 1.0 / growth, z)
    torch.cuda.synchronize()
    got = z.cpu().numpy()
    for k in range(3):
        ref = reference(r[k].astype(np.float64), n)
        assert np.abs(got[k, :n - 1, :n - 1] - ref).max() <= 4e-3 * np.abs(ref).max(), k
        assert not got[k, n - 1].any() and not got[k, :, n - 1].any()


@pytest.mark.parametrize("n,prec,margin", [(128, 0, 1.05), (256, 0, 1.05), (256, 1, 1.1)])
def test_iterations_on_rough_fields(n, prec, margin):
    """Only the observations wanted, a solve takes the iterations of one that keeps its solution (whose step
    lengths come from r.z in 64 bits): on smooth fields to one, on fields without decay, where hundreds show
    a loss of conjugacy, to 5 % on average; in FP32, which starts from another direction, to 10 %."""
    from paper_2503_16028_amd import smc
    N = 64
    d = json.load(open(golden("problem_t2.json")))
    d.update(grids=[n], kl_per_axis=32)
    p = smc.Problem(d, N, max_iter=2000)
    k = np.arange(32.0) ** 2
    flat = (1 + np.pi ** 2 * (k[:, None] + k)).reshape(-1) / 32
    for name, x in (("smooth", inputs.particles(N, p.K, 7)), ("rough", inputs.particles(N, p.K, 8) * flat)):
        print("[case] iterations", n, prec, name, flush=True)
        xi = torch.tensor(x, device=DEV)
        G = torch.empty(N, p.n_obs, dtype=torch.float64, device=DEV)
        w = torch.empty(N, n * n, dtype=torch.float64, device=DEV)
        obs, kept = (torch.zeros(N, dtype=torch.int32, device=DEV) for _ in range(2))
        smc.smc_forward_batch(p, N, xi, None, prec, G, obs)
        smc.smc_forward_state(p, N, xi, prec, G, w, kept)
        torch.cuda.synchronize()
        assert smc.smc_status_flags(p) == 0
        o, q = obs.double().mean().item(), kept.double().mean().item()
        print("   ", o, q, flush=True)
        assert o <= (q + 1.0 if name == "smooth" else margin * q)


@pytest.mark.parametrize("n,prec,buffers", [(256, 1, 10), (256, 0, 4), (128, 0, 4)])
def test_directions_are_folded_within_a_sweep(n, prec, buffers):
    """A sweep with more iterations than there are direction buffers (ten in FP32, four in FP64) folds them into the
    correction on the way.  In FP32, which solves to 1e-3 a sweep, that takes a field without decay (of standard
    deviation about a half), even with an inner tolerance out of reach: smooth fields take six.  The counters show that one did: more iterations than buffers times the sweeps that
    iterated (each solve's last sweep only finds that it has converged).  Observations to 1e-9, as that solver's other
    tests have them."""
    from oracle.forward import observe, solve
    from oracle.problem import Problem as OProblem, synthesize
    from paper_2503_16028_amd import smc
    print("[case] folded directions", n, prec, flush=True)
    d = json.load(open(golden("problem_t2.json")))
    at = [[1, 1], [n // 2, n // 2], [n - 1, n // 4], [n // 3, n - 1]]
    d.update(grids=[n], obs_den=n, obs=at, y=[0.0] * 4, sigma=1.0)
    op = OProblem(d)
    N = 2
    p = smc.Problem(d, N, tol_inner=1e-14 if prec else 1e-3, max_iter=2000)
    x = inputs.particles(N, op.K, 64)
    if prec:
        k = np.arange(8.0) ** 2   # eight modes per axis
        x *= (1 + np.pi ** 2 * (k[:, None] + k)).reshape(-1) / 16
    G = torch.empty(N, 4, dtype=torch.float64, device=DEV)
    smc.smc_profile(p, True)
    smc.smc_forward_batch(p, N, torch.tensor(x, device=DEV), None, prec, G)
    c = smc.smc_profile_read(p)
    assert smc.smc_status_flags(p) == 0
    print("   ", c, flush=True)
    assert c["solves"] == N and c["iters"] > buffers * (c["sweeps"] - c["solves"])
    for k in range(N):
        ref = observe(op, solve(op, synthesize(op, x[k], n), n), n)
        assert np.abs(G[k].cpu().numpy() - ref).max() <= 1e-9 * np.abs(ref).max()
