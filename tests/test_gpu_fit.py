"""The mixture fit at the edges of its layout (columns per workgroup of the M-step, components per wave,
partials per thread, a ragged last tile) against the oracle, with the bounds of the other fit tests
(1e-9), and from the rows and from the gathered tiles to the same bits."""
import sys

import numpy as np
import pytest
import torch

import inputs
from oracle import gmfit

pytestmark = pytest.mark.gpu
DEV = "cuda"


def t(a, dtype=torch.float64):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device=DEV)


@pytest.mark.parametrize("N,K,kr,M,iters", [
    (1, 3, 1, 1, 2), (63, 40, 15, 2, 6), (64, 20, 16, 4, 6), (65, 64, 30, 5, 6), (2049, 33, 31, 9, 6),
    (4097, 64, 46, 16, 5), (20001, 64, 64, 8, 4)])
def test_fit_edges(N, K, kr, M, iters):
    from paper_2503_16028_amd import smc
    print("[case] fit edges", N, K, kr, M, iters, flush=True)
    sys.stdout.flush()
    p = smc.L2MixProblem(K, kr, 0.01, np.zeros((1, K)), 1.0, N)      # the first kr modes are active
    xi = inputs.particles(N, K, 5)
    xi[:, :kr] = inputs.clusters(N, kr, M, 6, sep=4.0)[0]
    out = []
    for which in ("problem", "rows"):
        logw = torch.empty(M, dtype=torch.float64, device=DEV)
        mean, scale = (torch.empty(M, kr, dtype=torch.float64, device=DEV) for _ in range(2))
        cen = torch.empty(M, dtype=torch.int32, device=DEV)
        if which == "problem":
            smc.smc_gm_fit(p, N, t(xi), M, iters, 1e-3, 7, 70, logw, mean, scale, cen)
        else:
            smc.smc_gm_fit_noalloc(N, K, t(np.arange(kr), torch.int32), t(xi), M, iters, 1e-3, 7, 70, logw, mean, scale,
                                   cen)
        out.append((logw, mean, scale, cen))
    assert all(torch.equal(a, b) for a, b in zip(*out))
    rc, info = gmfit.kmeanspp_philox(xi[:, :kr], M, 7, 70, margins=True)
    assert all(mg > bound and clear for mg, bound, clear in info) and out[0][3].tolist() == rc
    rlogw, rmean, rvar = gmfit.em(xi[:, :kr], *gmfit.start(xi[:, :kr], rc), iters)
    logw, mean, var = (a.cpu().numpy() for a in out[0][:3])
    assert np.abs(logw - rlogw).max() <= 1e-9 * max(1.0, np.abs(rlogw).max())
    assert np.abs(mean - rmean).max() <= 1e-9 * max(1.0, np.abs(rmean).max())
    assert np.abs(var / rvar - 1).max() <= 1e-9
