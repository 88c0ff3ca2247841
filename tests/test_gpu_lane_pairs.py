"""Lane kernels with propensities in the pair form (networks of three to eight species,
at most eight reactions of at most two molecules): sources, conversions, pairs of
equal and of different molecules, counts at 0, 1 and 2 where a pair's propensity
vanishes, all eight species and reactions used, and a third-order network beside
them, which keeps the general form, as two species do.  Bit for bit the CPU oracle's
ensembles."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _net(S, third=False):
    n = [f"X{i}" for i in range(S)]
    last = n[-1]
    rx = [({}, {n[0]: 1}, 6.0), ({n[0]: 1}, {n[1]: 1}, 1.1), ({n[1]: 2}, {last: 2}, 0.7),
          ({n[0]: 1, n[1]: 1}, {n[0]: 2}, 0.3), ({last: 1}, {}, 0.9)]
    if S > 2:
        rx += [({n[i]: 1, n[0]: 1}, {n[i - 1]: 1, last: 1}, 0.2 + 0.1 * i) for i in (2, S - 1)]
        rx += [({n[2]: 1}, {n[S // 2]: 1}, 0.5)]
    if third:
        rx[-1] = ({n[0]: 3}, {n[0]: 2}, 0.05)
    return wl.Network.from_reactions(n, rx)


@pytest.mark.parametrize("S,third,x0", [(2, False, 0), (2, False, 1), (2, True, 3), (3, False, 2), (6, False, 1), (7, False, 4),
                                        (8, False, 0), (8, False, 2), (8, True, 3)])
def test_small_networks(S, third, x0):
    print(f"case: lane pairs, {S} species, third order {third}, from {x0}", flush=True)
    from paper_1303_5986_amd import we
    coef = np.zeros(S)
    coef[0], coef[-1] = 1.0, 0.5
    cfg = wl.WEConfig(name="pairs", net=_net(S, third), x0=np.full(S, x0, np.int32), bin_coef=coef,
                      edges=wl.uniform_edges(0.0, 24.0, 12), m_targ=12, tau=0.5, n_iters=6,
                      seeds=np.arange(11, 14, dtype=np.uint64))
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=6)
    ors = [orc.OracleWE(cfg, int(s)) for s in cfg.seeds]
    for it in range(6):
        sim.step(1)
        for r, o in enumerate(ors):
            o.step(1)
            for g, e, what in zip(sim.walkers(r), o.walkers(), ("counts", "weights", "bins", "parents")):
                assert np.array_equal(np.asarray(g).view(np.uint8), np.asarray(e).view(np.uint8)), (it, r, what)
    assert sum(sum(o.events) for o in ors) > 0
