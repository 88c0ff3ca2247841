"""The work queue's order kernel at the edges of its forms: one launch (up to
4096 segments and 1024 counters) and three, one and several threads per bin, one
replica of the counters and 128, few bins and more than 1024.  A walker that the
queue lost, listed twice or gave a wrong slot would differ from the CPU oracle:
counts, weights, bins and parents must be equal bit for bit."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl

# name: (bins, width of a bin, walkers per bin, runs)
CASES = {
    "2 bins": (2, 45.0, 5, 40),
    "4096 segments, one launch": (64, 3.0, 4, 64),
    "4160 segments, three": (65, 3.0, 4, 64),
    "1024 counters, one launch": (1024, 1.0, 2, 3),
    "1025 counters, three": (1025, 1.0, 2, 3),
    "513 bins, one thread each": (513, 1.0, 3, 40),
    "100 bins, 16 replicas": (100, 2.0, 3, 260),
    "5 bins, 128 replicas": (5, 25.0, 3, 2100),
    "129 bins, 127 replicas": (129, 2.0, 2, 2050),
    "7700 bins": (7700, 0.25, 1, 2),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_every_walker_is_queued_once(name):
    print(f"case: queue order, {name}", flush=True)
    from paper_1303_5986_amd import we
    nb, width, m, runs = CASES[name]
    base = wl.schlogl_config(n_runs=runs, seed0=77, n_iters=5)
    cfg = dataclasses.replace(base, name="queue", m_targ=m, tau=0.1, edges=wl.uniform_edges(0.0, nb * width, nb),
                              tgt_thr=130.0)
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=5)
    ors = {r: orc.OracleWE(cfg, int(cfg.seeds[r])) for r in sorted({0, runs // 3, runs // 2, runs - 1})}
    for it in range(5):
        sim.step(1)
        for r, o in ors.items():
            o.step(1)
            for g, e, what in zip(sim.walkers(r), o.walkers(), ("counts", "weights", "bins", "parents")):
                assert np.array_equal(np.asarray(g).view(np.uint8), np.asarray(e).view(np.uint8)), (it, r, what)
