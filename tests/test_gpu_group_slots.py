"""Group kernels with as many register slots as a lane's block of reactions needs:
blocks of 1, 2, 3, 4, 5 and 8 reactions, with the last lanes' blocks shorter or
empty.  Walkers against the CPU oracle, of which at most 1% may differ (an event
changes only where rounding of another summation order decides it)."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _ring(S, R):
    n = [f"X{i}" for i in range(S)]
    rx = [({}, {n[0]: 1}, 5.0), ({n[0]: 2}, {n[1]: 1}, 0.3)]
    while len(rx) < R:
        i = len(rx)
        rx.append(({n[i % S]: 1}, {n[(i + 1) % S]: 1}, 0.5 + 0.05 * i) if i % 3 else
                  ({n[i % S]: 1, n[(i + 2) % S]: 1}, {n[(i + 1) % S]: 1}, 0.02 * i))
    return wl.Network.from_reactions(n, rx)


@pytest.mark.parametrize("wpw,R", [(8, 8), (8, 9), (8, 16), (8, 17), (8, 31), (8, 33), (16, 7), (16, 12), (4, 20), (4, 64),
                                   (2, 40), (32, 4), (32, 15)])
def test_blocks_of_reactions(wpw, R):
    print(f"case: group slots, {wpw} walkers per wave, {R} reactions", flush=True)
    from paper_1303_5986_amd import we
    coef = np.zeros(5)
    coef[1] = 1.0
    cfg = wl.WEConfig(name="ring", net=_ring(5, R), x0=np.full(5, 6, np.int32), bin_coef=coef,
                      edges=wl.uniform_edges(0.0, 16.0, 8), m_targ=8, tau=0.3, n_iters=8,
                      seeds=np.arange(21, 24, dtype=np.uint64))
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_GROUP, walkers_per_wave=wpw, max_iters=8)
    sim.step(8)
    total = same = fired = 0
    for r, s in enumerate(cfg.seeds):
        o = orc.OracleWE(cfg, int(s))
        o.step(8)
        x, w, _, _ = sim.walkers(r)
        ox, ow, _, _ = o.walkers()
        total += len(ow)
        fired += sum(o.events)
        if len(w) == len(ow):
            same += int(((x == ox).all(axis=1) & (w == ow)).sum())
    assert fired > 1000 and same >= 0.99 * total, (same, total)
