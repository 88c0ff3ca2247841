"""Propensities so small that their reciprocal is past the range of a double: the
next event lies past any interval, so nothing fires, as in the oracle.  Every
kernel family, alone and in a batch; beside a rate in the normal range that runs out,
after which only the tiny ones are left."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl

pytestmark = pytest.mark.gpu

LANE, WAVE, GROUP = 1, 2, 3


def _config(S, extra, rate, hill=False, engine="ssa"):
    """X0 decays at an ordinary rate; conversions at `rate` never happen."""
    n = [f"X{i}" for i in range(S)]
    rx = [({n[0]: 1}, {}, 30.0)]
    if S == 1:
        rx += [({n[0]: 2}, {n[0]: 3}, rate), ({}, {n[0]: 1}, rate)]
    for i in range(1, S):
        rx += [({n[i]: 1}, {n[i % (S - 1) + 1]: 1} if S > 2 else {n[i]: 2}, rate)]
    for j in range(extra):
        rx += [({n[j % S]: 1, n[(j + 1) % S]: 1}, {n[(j + 2) % S]: 2}, rate) if S > 1 else ({n[0]: 3}, {}, rate)]
    if hill:
        rx[1] = (*rx[1], (n[0], 2, 5.0))
    coef = np.zeros(S)
    coef[0] = 1.0
    return wl.WEConfig(name="tiny", net=wl.Network.from_reactions(n, rx), x0=np.full(S, 2, np.int32), bin_coef=coef,
                       edges=wl.uniform_edges(0.0, 4.0, 4), m_targ=12, tau=1.0, n_iters=3,
                       seeds=np.arange(3, 5, dtype=np.uint64), engine=engine)


@pytest.mark.parametrize("S,extra,kernel,wpw", [(1, 0, LANE, 0), (2, 2, LANE, 0), (5, 1, LANE, 0), (7, 6, LANE, 0),
                                                (12, 10, LANE, 0), (25, 20, LANE, 0), (6, 40, GROUP, 8), (6, 70, GROUP, 32),
                                                (20, 100, WAVE, 0), (600, 100, WAVE, 0)])
@pytest.mark.parametrize("rate", [5e-324, 1e-310, 2e-309])
def test_nothing_fires(S, extra, kernel, wpw, rate):
    from paper_1303_5986_amd import we
    print(f"case: rates of {rate}, {S} species, kernel {kernel}", flush=True)
    cfg = _config(S, extra, rate)
    sim = we.sim_from_config(cfg, kernel=kernel, walkers_per_wave=wpw, max_iters=3)
    sim.step(3)
    b = we.Batch([cfg], max_iters=3, kernels=[(kernel, wpw) if wpw else kernel])
    b.step(3)
    for r, s in enumerate(cfg.seeds):
        o = orc.OracleWE(cfg, int(s))
        o.step(3)
        for got in (sim.walkers(r), b.members[0].walkers(r)):
            assert (got[0][:, 1:] == 2).all()
            for g, e in zip(got, o.walkers()):
                assert np.array_equal(g, e), r


@pytest.mark.parametrize("S,extra,hill,engine", [(2, 0, True, "ssa"), (4, 0, True, "ssa"), (1, 0, False, "tauleap"),
                                                 (2, 2, False, "tauleap"), (7, 5, False, "tauleap")])
def test_nothing_fires_hill_and_leaps(S, extra, hill, engine):
    from paper_1303_5986_amd import we
    print(f"case: rates of 1e-310, {S} species, Hill {hill}, {engine}", flush=True)
    cfg = _config(S, extra, 1e-310, hill, engine)
    sim = we.sim_from_config(cfg, kernel=LANE, max_iters=3)
    sim.step(3)
    for r, s in enumerate(cfg.seeds):
        o = orc.OracleWE(cfg, int(s))
        o.step(3)
        for g, e in zip(sim.walkers(r), o.walkers()):
            assert np.array_equal(g, e), r
