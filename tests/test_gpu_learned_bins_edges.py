"""Learned bins where the binning kernel's parts end: walker numbers that leave a
group of four unfilled, edges counted in one and several passes of 64, and the
binary search past 256 bins.  Every live walker sits in the oracle's bin of its
FP64 logit on the caller's edges; within 1e-3 of an edge the FP32 logit may fall
on the other side and either neighbour is accepted."""
import dataclasses

import numpy as np
import pytest

from oracle import mlp
from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,m", [(2, 5), (64, 3), (65, 7), (66, 2), (256, 3), (257, 3)])
def test_bins_on_caller_edges(nb, m):
    print(f"case: learned bins, {nb} bins of {m}", flush=True)
    from paper_1303_5986_amd import we
    base = wl.toggle_config(n_runs=3, n_iters=24)
    lo, hi = float(base.edges[0]), float(base.edges[-1])
    cfg = dataclasses.replace(base, m_targ=m, edges=wl.uniform_edges(lo, hi, nb))
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=24, record_iters=20)
    sim.step(20)
    sim.train_committor(cfg.bin_coef, base.a_thr, steps=50, batch=256, lr=2e-3, seed=5, edge_mode=1)
    e = np.linspace(-3.0, 3.0, nb + 1)
    sim.set_learned_bins(e)
    sim.step(3)
    p, feat, _ = sim.committor_state()
    seen = 0
    for r in range(3):
        x, w, b, _ = sim.walkers(r)
        _, _, _, z = mlp.forward(p.astype(np.float64), feat.astype(np.float64), x, cfg.net.S)
        ref = np.array([orc.bin_of(e, float(v)) for v in z])
        near = np.min(np.abs(z[:, None] - e[None, 1:-1]), axis=1) <= 1e-3
        assert np.array_equal(b[~near], ref[~near])
        assert np.all(np.abs(b[near] - ref[near]) <= 1)
        seen += int(np.sum(~near))
    assert seen > 0
