"""Placement of walkers by bin: one bin, numbers of bins around powers of two
(a ballot per bit of the bin's number), more bins than cursor rows for all
waves, more walkers than a pass of the recycled sum takes (512), and few walkers
in a last chunk; recycled and binned beforehand or by the run's workgroup (one walker
per thread at most); with the bins merged in the run's workgroup and by bin, for
both rules.  Everything against the CPU oracle, bit for bit."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl

# name: (bins, width of a bin, walkers per bin, runs, rule, recycled above)
CASES = {
    "one bin": (1, 800.0, 70, 2, 0, 90),
    "two bins": (2, 45.0, 33, 2, 1, 100),
    "three bins": (3, 30.0, 64, 1, 0, 95),
    "33 bins by bin": (33, 4.0, 20, 3, 0, 110),
    "64 bins by bin": (64, 2.0, 9, 2, 1, 108),
    "65 bins by bin": (65, 2.0, 40, 2, 0, 104),
    "513 bins by bin": (513, 1.0, 11, 2, 0, 102),
    "1100 bins, 7 rows": (1100, 1.0, 5, 1, 1, 101),
    "6000 bins, one row": (6000, 1.0, 3, 1, 0, 99),
    "many runs": (17, 10.0, 12, 520, 0, 95),
    "a walker per thread": (16, 8.0, 64, 2, 0, 95),
    "some threads two": (16, 8.0, 65, 2, 1, 95),
    "many runs, a walker per thread": (16, 8.0, 16, 512, 1, 95),
    "many runs, some threads two": (16, 8.0, 17, 512, 0, 95),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_placement_matches_oracle(name):
    print(f"case: placement, {name}", flush=True)
    from paper_1303_5986_amd import we
    nb, width, m, runs, rule, thr = CASES[name]
    base = wl.schlogl_config(n_runs=runs, seed0=31, n_iters=6)
    cfg = dataclasses.replace(base, name="place", m_targ=m, tau=0.1, edges=wl.uniform_edges(0.0, nb * width, nb),
                              tgt_thr=float(thr), resample_rule=rule)
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=6)
    checked = range(runs) if runs < 8 else (0, 255, runs - 1)
    ors = {r: orc.OracleWE(cfg, int(cfg.seeds[r])) for r in checked}
    recycled = 0.0
    for it in range(6):
        sim.step(1)
        for r, o in ors.items():
            o.step(1)
            for g, e, what in zip(sim.walkers(r), o.walkers(), ("counts", "weights", "bins", "parents")):
                assert np.array_equal(np.asarray(g).view(np.uint8), np.asarray(e).view(np.uint8)), (it, r, what)
            assert np.array_equal(sim.flux(r), o.flux), (it, r)
            recycled += float(np.sum(o.flux))
    assert recycled > 0.0
