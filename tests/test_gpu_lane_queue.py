"""The lane kernels' work queue over several heads: every walker is propagated
exactly once whatever the number of queue segments, from one segment to more
tiles than static first positions, with segment lengths that do not divide a
tile of 64 positions and walker counts on both sides of the heads' and blocks'
thresholds.  Each sim's ensembles equal the oracle's bit for bit (one run of
many is compared where there are many)."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("runs,bins,m", [(1, 1, 1), (1, 7, 3), (2, 20, 13), (31, 13, 5), (33, 60, 65), (300, 60, 8),
                                         (2100, 30, 11)])
def test_every_walker_once(runs, bins, m):
    from paper_1303_5986_amd import we
    print(f"case: lane queue runs={runs} bins={bins} m={m}", flush=True)
    cfg = dataclasses.replace(wl.birth_death_config(n_runs=runs, seed0=9), m_targ=m,
                              edges=wl.uniform_edges(0.0, 120.0, bins))
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=6)
    sim.step(6)
    for r in sorted({0, runs // 2, runs - 1}):
        o = orc.OracleWE(cfg, int(cfg.seeds[r]))
        o.step(6)
        x, w, b, _ = sim.walkers(r)
        ox, ow, ob, _ = o.walkers()
        assert np.array_equal(x, ox) and np.array_equal(w, ow) and np.array_equal(b, ob), r
        assert np.array_equal(sim.flux(r), np.array(o.flux)), r
