"""The lane kernels' teams: when a wave's last walkers are spread over several
lanes each, whatever their number (1 to 64 per wave, walkers that end at very
different events), on every variant that has them (one species, two species,
up to eight species, Hill-type rates), with recycling, and at the edges of an
interval (no event at all, no reaction possible).  Bit for bit the oracle's
ensembles."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _schlogl(n, tau):
    c = dataclasses.replace(wl.schlogl_config(n_runs=1, seed0=21), tau=tau, m_targ=1,
                            edges=wl.uniform_edges(0.0, 800.0, n))
    x = np.linspace(2, 790, n).astype(np.int32)[:, None]     # one walker per bin, 30 to 20000 events per unit time
    return c, x


def _case(name):
    if name.startswith("schlogl"):
        return _schlogl(int(name[7:]), 0.02)
    if name == "quiet":          # fewer than one event per interval
        return _schlogl(40, 1e-5)
    if name == "dying":          # 2X -> 0 and X -> 0 only: walkers run out of molecules
        net = wl.Network.from_reactions(["X"], [({"X": 2}, {}, 0.5), ({"X": 1}, {}, 0.1)])
        c = wl.WEConfig(name="dying", net=net, x0=np.array([0], np.int32), bin_coef=np.array([1.0]),
                        edges=wl.uniform_edges(0.0, 60.0, 30), m_targ=2, tau=5.0, n_iters=0,
                        seeds=np.array([4], np.uint64))
        return c, np.arange(60, dtype=np.int32)[:, None]
    if name == "switch":
        c = dataclasses.replace(wl.switch_config(n_runs=1, seed0=6, m_targ=2))
        r = np.random.default_rng(3)
        return c, np.stack([r.integers(0, 160, 200), r.integers(0, 32, 200)], axis=1).astype(np.int32)
    r = np.random.default_rng(5)
    S, R = (2, 6) if name == "two" else (6, 14)
    net = wl.random_network(40 + S, S, R, rate_lo=0.05, rate_hi=2.0)
    coef = np.zeros(S)
    coef[0] = 1.0
    c = wl.WEConfig(name=name, net=net, x0=np.full(S, 5, np.int32), bin_coef=coef, edges=wl.uniform_edges(0.0, 200.0, 40),
                    m_targ=3, tau=0.5, n_iters=0, seeds=np.array([8], np.uint64))
    return c, (10.0 ** r.uniform(0, 2.3, (100, S))).astype(np.int32)


@pytest.mark.parametrize("name", ["schlogl1", "schlogl2", "schlogl31", "schlogl33", "schlogl64", "schlogl65",
                                  "schlogl300", "quiet", "dying", "two", "six", "switch"])
def test_teams_match_oracle(name):
    from paper_1303_5986_amd import we
    print(f"case: lane teams {name}", flush=True)
    cfg, x = _case(name)
    w = np.full(len(x), 1.0 / len(x))
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=5)
    sim.set_ensemble(0, x, w)
    o = orc.OracleWE(cfg, int(cfg.seeds[0]), init_x=x, init_w=w)
    for it in range(5):
        sim.step(1)
        o.step(1)
        for a, c in zip(sim.walkers(0), o.walkers()):
            assert np.array_equal(a, c), it
    assert np.array_equal(sim.flux(0, 0, 5), np.array(o.flux))
