"""Device memory a problem holds (GPU): its workspace is for moves and fits of n_max particles, and a fit's copy of
the cloud shares the proposal rows."""
import sys

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("n_max,K,kr", [(1 << 20, 64, 64), (1 << 19, 64, 16)])
def test_memory_of_a_problem(n_max, K, kr):
    from paper_2503_16028_amd import smc
    print("[case] workspace", n_max, K, kr, flush=True)
    sys.stdout.flush()
    smc.L2MixProblem(K, kr, 0.01, np.zeros((1, K)), 0.3, 64).close()   # code and tables are loaded
    before = free_bytes()
    p = smc.L2MixProblem(K, kr, 0.01, np.zeros((1, K)), 0.3, n_max)
    held = before - free_bytes()
    # a row of proposals, the log ratio, the new potential, the iterations and the seeding distance of each
    # particle, and the partial sums of the fit, 16 components of 1 + 2 * 64 values for every 64 particles
    want = n_max * (8 * K + 8 + 8 + 4 + 8) + (n_max + 63) // 64 * 16 * 129 * 8
    assert held <= want + (32 << 20)
    p.close()


@pytest.mark.parametrize("N", [64, 65, 1000])
def test_fit_leaves_the_neighbours_alone(N):
    """The tiles end on whole groups of 64 particles, past the rows of an odd cloud of all its modes: a problem sized
    to the cloud fits it as a larger one does, between moves that use the same rows."""
    from paper_2503_16028_amd import smc
    K, M = 8, 3
    f64 = dict(dtype=torch.float64, device=DEV)
    g = torch.Generator(device=DEV).manual_seed(N)
    c = np.linspace(-1.0, 1.0, K)[None]
    xi0 = torch.randn(N, K, generator=g, **f64)
    gm = (torch.zeros(1, **f64), torch.zeros(1, K, **f64), torch.ones(1, K, **f64))
    got = []
    for n_max in (N, 4 * N):
        p = smc.L2MixProblem(K, K, 0.01, c, 0.3, n_max)
        xi, phi = xi0.clone(), torch.empty(N, **f64)
        acc = torch.empty(N, dtype=torch.int32, device=DEV)
        fit = [torch.empty(M, **f64), torch.empty(M, K, **f64), torch.empty(M, K, **f64)]
        smc.smc_phi_batch(p, N, xi, None, smc.SMC_FP64, phi)
        smc.smc_gmpcn_move(p, N, gm, 0.4, 0.5, 3, 1, 100, None, smc.SMC_FP64, xi, phi, acc)
        smc.smc_gm_fit(p, N, xi, M, 10, 1e-3, 2, 7, *fit)
        smc.smc_gmpcn_move(p, N, gm, 0.4, 0.5, 3, 1, 200, None, smc.SMC_FP64, xi, phi, acc)
        torch.cuda.synchronize()
        assert smc.smc_status_flags(p) == 0
        got.append([a.clone() for a in (xi, phi, acc, *fit)])
    assert all(torch.equal(a, b) for a, b in zip(*got))
