"""Reweighting events over wide components: a component across the 64-state
chunks, rows longer than one pass of an elimination step (256 entries) and as
many bins as are taken (512), in LDS and in device memory; bins of one walker
and of many.  The flux matrix itself, with bins of fewer and more than 64 walkers
from many start bins, equals the oracle's bit for bit.  The event is recomputed on the host from the flux matrix and the
weights of a twin that skips it: state reduction in extended precision on the
same strongly connected component.  State reduction in FP64 has an entrywise
relative error of order n^3 u (O'Cinneide 1993): rtol = n^3 u, n the component's
size; walkers outside the component keep their weights bit for bit."""
import numpy as np
import pytest
from scipy.sparse import csr_matrix
from scipy.sparse.csgraph import connected_components

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl

U = 2.0 ** -53


def expected(F, b, w):
    """-> (factor per bin, component size)"""
    nb = F.shape[0]
    wb = np.bincount(b, weights=w, minlength=nb)
    W = F.sum(axis=0)
    cand = np.flatnonzero((wb > 0) & (W > 0))
    fac = np.ones(nb)
    if len(cand) < 2:
        return fac, 0
    A = (F[np.ix_(cand, cand)] > 0)
    label = connected_components(csr_matrix(A), directed=True, connection="strong")[1]
    comp = cand[label == label[np.argmax(wb[cand])]]
    n = len(comp)
    if n < 2:
        return fac, n
    R = (F[np.ix_(comp, comp)].T / W[comp][:, None]).astype(np.longdouble)   # from, to
    np.fill_diagonal(R, 0)
    s = np.zeros(n, np.longdouble)
    for m in range(n - 1, 0, -1):
        s[m] = R[m, :m].sum()
        R[:m, :m] += np.outer(R[:m, m], R[m, :m] / s[m])
        R[np.arange(m), np.arange(m)] = 0
    pi = np.zeros(n, np.longdouble)
    pi[0] = 1
    for m in range(1, n):
        pi[m] = (pi[:m] * R[:m, m]).sum() / s[m]
    fac[comp] = (pi / pi.sum() * wb[comp].sum() / wb[comp]).astype(np.float64)
    return fac, n


def bursts(size, burst_rate, decay):
    """0 -> size X, X -> 0: a wide stationary distribution, jumps over many bins."""
    return wl.Network.from_reactions(["X"], [({}, {"X": size}, burst_rate), ({"X": 1}, {}, decay)])


# name: (bins, width of a bin, walkers per bin, (size, rate, decay), tau, interval of the
#        event, component size at least)
CASES = {
    "two bins": (2, 40.0, 3, (1, 40.0, 1.0), 1.0, 4, 2),
    "64 states": (64, 4.0, 40, (8, 16.0, 1.0), 0.5, 8, 33),
    "65 bins, far jumps": (65, 4.0, 16, (40, 6.0, 1.0), 1.0, 12, 49),
    "129 bins": (129, 2.0, 16, (40, 6.0, 1.0), 1.0, 12, 97),
    "300 bins, far jumps": (300, 1.6, 12, (60, 5.0, 1.0), 1.0, 14, 257),
    "as many as are taken": (512, 0.9, 8, (60, 5.0, 1.0), 1.0, 14, 353),
}


def _cfg(name):
    nb, width, m, net, tau, n, _ = CASES[name]
    return wl.WEConfig(name="wide", net=bursts(*net), x0=np.array([40], np.int32), bin_coef=np.array([1.0]),
                       edges=wl.uniform_edges(0.0, nb * width, nb), m_targ=m, tau=tau, n_iters=n,
                       seeds=np.array([5, 6], np.uint64))


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_event_over_wide_components(name):
    print(f"case: wide reweighting, {name}", flush=True)
    from paper_1303_5986_amd import we
    cfg = _cfg(name)
    n = CASES[name][5]
    sims = [we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=n, rw_period=p) for p in (n, n + 1)]
    for s in sims:
        s.step(n)
    for r in range(2):
        x, w, b, o = sims[0].walkers(r)
        x1, w1, b1, o1 = sims[1].walkers(r)
        F = sims[0].rw_flux_matrix(r)
        assert np.array_equal(x, x1) and np.array_equal(b, b1) and np.array_equal(o, o1)
        assert np.array_equal(F, sims[1].rw_flux_matrix(r))
        fac, size = expected(F, b, w1)
        assert size >= CASES[name][6]
        assert sims[0].rw_counts(r) == ((1, 0) if size >= 2 else (0, 1))
        assert np.array_equal(w[fac[b] == 1.0], w1[fac[b] == 1.0])
        np.testing.assert_allclose(w, w1 * fac[b], rtol=max(size, 2) ** 3 * U, atol=0)
        print(f"run {r}: component of {size}", flush=True)


@pytest.mark.gpu
@pytest.mark.parametrize("nb,width,m", [(33, 8.0, 17), (64, 6.0, 64), (65, 6.0, 90), (20, 15.0, 150)])
def test_flux_matrix_of_large_bins_is_the_oracles(nb, width, m):
    print(f"case: flux matrix, {nb} bins of {m}", flush=True)
    from paper_1303_5986_amd import we
    cfg = wl.WEConfig(name="flux", net=bursts(40, 6.0, 1.0), x0=np.array([40], np.int32), bin_coef=np.array([1.0]),
                      edges=wl.uniform_edges(0.0, nb * width, nb), m_targ=m, tau=0.6, n_iters=6,
                      seeds=np.array([3, 4], np.uint64))
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=6, rw_period=7)
    sim.step(6)
    for r in range(2):
        o = orc.OracleWE(cfg, int(cfg.seeds[r]), rw_period=7)
        o.step(6)
        assert np.array_equal(sim.rw_flux_matrix(r), o.rw_F), r
        assert np.count_nonzero(o.rw_F) > 2 * nb
