"""Re-weighting, resampling and gather at the edges of their launches: one workgroup and many, whole and
ragged tiles and chunks, a search that outlasts the launched passes (stall), weights written over the potentials,
outputs on odd addresses, every row width.  Against the oracle with the bounds of the other tests of
these calls: 1e-10 for the increment and the weights, exact indices and rows."""
import sys

import numpy as np
import pytest
import torch

import inputs
from oracle.resample import systematic
from oracle.temper import temper

pytestmark = pytest.mark.gpu
DEV = "cuda"


def banner(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


def t(a, dtype=torch.float64):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device=DEV)


def potentials(N, kind):
    rng = np.random.default_rng(N)
    if kind == "wide":                       # a search of about eleven passes
        return np.exp(12.0 * rng.standard_normal(N) + 4.0)
    if kind == "stall":
        p = np.full(N, 1e308)
        p[N // 2] = 0.0
        return p
    p = inputs.potentials(N, N)
    if kind == "holes":
        p[rng.random(N) < 0.4] = np.inf
        p[0] = p[-1] = np.nan
    if kind == "none":
        p[:] = np.nan
    return p


@pytest.mark.parametrize("N,kind,place", [
    (255, "plain", "apart"), (8064, "plain", "apart"), (8065, "plain", "apart"), (8065, "plain", "over"),
    (9001, "wide", "apart"), (9001, "stall", "apart"), (9001, "none", "apart"), (9001, "holes", "odd"),
    (262145, "holes", "apart"), (300001, "plain", "odd"), (1 << 20, "holes", "over")])
def test_temper_launches(N, kind, place):
    from paper_2503_16028_amd import smc
    banner("temper", N, kind, place)
    phi0 = potentials(N, kind)
    room = torch.full((2 * N + 3,), 7.0, dtype=torch.float64, device=DEV)
    phi = room[1:N + 1] if place == "odd" else room[:N]
    phi.copy_(t(phi0))
    W = phi if place == "over" else room[N + 1:2 * N + 1]
    h, tau_new, lz = (torch.empty(1, dtype=torch.float64, device=DEV) for _ in range(3))
    flags = torch.zeros(1, dtype=torch.int32, device=DEV)
    smc.smc_temper(N, phi, t([0.1]), 0.5, h, tau_new, W, lz, flags)
    Wg = W.cpu().numpy()
    if kind == "none":
        assert h.item() == 0.0 and tau_new.item() == 0.1 and lz.item() == -np.inf
        assert not Wg.any() and flags.item() == smc.FLAG_NONFINITE
        return
    rh, rtau, rW, rlz, stalled = temper(phi0, 0.1, 0.5)
    assert flags.item() == (smc.FLAG_STALL if stalled else 0)
    assert h.item() == pytest.approx(rh, rel=1e-10, abs=1e-300) and tau_new.item() == pytest.approx(rtau, rel=1e-12)
    assert lz.item() == pytest.approx(rlz, rel=1e-10, abs=1e-10)
    pos = rW > 1e-290
    assert np.array_equal(Wg[rW == 0.0], rW[rW == 0.0]) and np.abs(Wg[pos] / rW[pos] - 1).max() <= 1e-10
    outside = [room[N + (place == "odd"):N + 1], room[2 * N + 1:]] if place != "over" else [room[N:]]
    assert all((o == 7.0).all() for o in outside)


@pytest.mark.parametrize("N", [8191, 8192, 8193, 10241, 100003, (1 << 20) + 1])
@pytest.mark.parametrize("kind", ["dirichlet", "first", "last", "few", "bad"])
def test_resample_launches(N, kind):
    from paper_2503_16028_amd import smc
    banner("resample", N, kind)
    W = inputs.weights(N, N + 3, "dirichlet")
    if kind in ("first", "last"):            # one end owns all but a sprinkling
        W *= 1e-3
        W[0 if kind == "first" else -1] += 1.0 - W.sum() - 1e-12
    if kind == "few":                        # one output here and there, in the first entries too
        W[:] = 0.0
        W[::N // 7] = 0.1
    if kind == "bad":
        W[N - 1] = np.nan
    u = inputs.u53(N)
    room = torch.full((N + 2,), -5, dtype=torch.int32, device=DEV)
    idx = room[1:N + 1]                      # 4-byte aligned only
    flags = torch.zeros(1, dtype=torch.int32, device=DEV)
    smc.smc_resample(N, t(W), u, idx, flags)
    want = np.arange(N) if kind == "bad" else np.array(systematic(W, u))
    assert np.array_equal(idx.cpu().numpy(), want) and room[0] == -5 and room[-1] == -5
    assert flags.item() == (smc.FLAG_BADWEIGHTS if kind == "bad" else 0)


@pytest.mark.parametrize("N,K", [(1, 1), (77, 17), (301, 32), (300, 66), (65, 130), (9, 258), (33, 1023), (66000, 34),
                                 (33001, 128), (270001, 1)])
@pytest.mark.parametrize("off", [0, 1])
def test_gather_widths(N, K, off):
    from paper_2503_16028_amd import smc
    banner("gather", N, K, off)
    rng = np.random.default_rng(K)
    ii = rng.integers(0, N, N)
    src, dst = (torch.full((N * K + 2,), 3.0, dtype=torch.float64, device=DEV) for _ in range(2))
    xi, xo = src[off:off + N * K].view(N, K), dst[off:off + N * K].view(N, K)
    xi.copy_(t(rng.standard_normal((N, K))))
    phi, po = t(rng.standard_normal(N)), torch.empty(N, dtype=torch.float64, device=DEV)
    idx = ii.copy()
    idx[N // 2] = N                          # out of range: the row stays
    smc.smc_gather(N, K, t(idx, torch.int32), xi, phi, xo, po)
    want = xi[t(ii, torch.int64)]
    want[N // 2] = 3.0
    keep = np.arange(N) != N // 2
    assert torch.equal(xo, want) and (dst[:off] == 3.0).all() and (dst[off + N * K:] == 3.0).all()
    assert np.array_equal(po.cpu().numpy()[keep], phi.cpu().numpy()[ii][keep])


def test_many_workgroups_in_a_graph():
    """The launch chains captured once and replayed on new potentials, eager calls in between: the same bits."""
    from paper_2503_16028_amd import smc
    banner("temper and resample chains in a graph")
    N = 20011
    phi, W = t(inputs.potentials(N, 1)), torch.empty(N, dtype=torch.float64, device=DEV)
    idx = torch.empty(N, dtype=torch.int32, device=DEV)
    tau = t([0.0])
    h, tau_new, lz = (torch.empty(1, dtype=torch.float64, device=DEV) for _ in range(3))
    u = inputs.u53(5)

    def both(W, idx, h, tau_new, lz):
        smc.smc_temper(N, phi, tau, 0.5, h, tau_new, W, lz)
        smc.smc_resample(N, W, u, idx)

    both(W, idx, h, tau_new, lz)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        both(W, idx, h, tau_new, lz)
    for r in range(3):
        phi.copy_(t(inputs.potentials(N, 10 + r)))
        tau.fill_(0.1 * r)
        g.replay()
        torch.cuda.synchronize()
        e = [torch.empty_like(a) for a in (W, idx, h, tau_new, lz)]
        both(*e)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(e, (W, idx, h, tau_new, lz))), r
        assert not torch.equal(idx, torch.arange(N, dtype=torch.int32, device=DEV))


@pytest.mark.parametrize("N", [64, 4096, 8064, 8065, 20000])
def test_next_double_does_not_pass(N):
    """The increment is the largest whose ESS passes, to a relative 2^-52: between 1/2 and 1 that is one double, and
    the call itself says so.  With tau = 1 - h the whole remaining step is h and passes (h and tau_new = 1 come
    back, both exact); with the next double in its place it does not."""
    from paper_2503_16028_amd import smc

    def step(phi, tau):
        h, tau_new, lz = (torch.empty(1, dtype=torch.float64, device=DEV) for _ in range(3))
        smc.smc_temper(N, phi, t([tau]), 0.5, h, tau_new, torch.empty(N, dtype=torch.float64, device=DEV), lz)
        return h.item(), tau_new.item()

    for seed in range(8):
        banner("next double", N, seed)
        phi0 = inputs.potentials(N, 100 + seed)
        h0, _ = step(t(phi0), 0.0)
        phi = t(phi0 * (h0 / (0.55 + 0.05 * seed)))
        h, _ = step(phi, 0.0)
        assert 0.5 < h < 1.0
        assert step(phi, 1.0 - h) == (h, 1.0)
        above = np.nextafter(h, 1.0)
        assert step(phi, 1.0 - above)[0] < above


@pytest.mark.parametrize("N", [4000, 8192, 8193, 100003, 1 << 20])
@pytest.mark.parametrize("heavy", [1, 3, 200])
def test_resample_few_heavy_particles(N, heavy):
    """Particles with many outputs each, alone and beside particles with few, written by their wave: exact, and in a
    time of the order of spread weights' (a thread by itself took a thousand times as long)."""
    from paper_2503_16028_amd import smc
    banner("resample heavy", N, heavy)
    rng = np.random.default_rng(N + heavy)
    W = inputs.weights(N, 5, "dirichlet") * 1e-2
    at = rng.choice(N, heavy, replace=False)
    at[0] = N // 2
    W[at] += 0.99 * (1 - 1e-9) / heavy
    u = inputs.u53(N)
    idx = torch.empty(N, dtype=torch.int32, device=DEV)
    smc.smc_resample(N, t(W), u, idx)
    assert np.array_equal(idx.cpu().numpy(), np.array(systematic(W, u)))
    spread = t(inputs.weights(N, 6, "dirichlet"))

    def best(w):
        out = np.inf
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        for _ in range(5):
            a.record()
            smc.smc_resample(N, w, u, idx)
            b.record()
            torch.cuda.synchronize()
            out = min(out, a.elapsed_time(b))
        return out

    few, many = best(t(W)), best(spread)
    print("   heavy %.3f ms, spread %.3f ms" % (few, many), flush=True)
    # a wave writes 64 outputs at a time: at most N / 64 stores in a row, 10 ns each on their way to memory
    assert few <= 2.0 * many + 0.02 + N / 64 * 1e-5
