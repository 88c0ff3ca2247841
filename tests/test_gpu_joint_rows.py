"""The joint histogram of rows that the observation itself copies (up to 16 species)
and of gathered ones (17), cell by cell: few and many runs, one to four species in
the histogram, cells shared by many walkers, counts past the last cell.  The
oracle's walkers give each cell's weights, which add up in another order (rtol n u
for the n of a run)."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl
from test_gpu_observe_rows import _chain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,runs,joint,bins,width", [
    (1, 2, [0], 8, 3), (8, 3, [0, 7], 6, 2), (8, 70, [7, 2, 0], 5, 2), (16, 2, [0, 15], 4, 1), (16, 66, [3, 9, 15, 0], 8, 1),
    (17, 3, [16, 0], 6, 2), (17, 65, [1, 16, 8], 7, 1)])
def test_cells(S, runs, joint, bins, width):
    print(f"case: joint histogram of species {joint} of {S}, {runs} runs", flush=True)
    from paper_1303_5986_amd import we
    coef = np.zeros(S)
    coef[-1] = 1.0
    cfg = wl.WEConfig(name="joint", net=_chain(S), x0=np.full(S, 3, np.int32), bin_coef=coef,
                      edges=wl.uniform_edges(0.0, 30.0, 15), m_targ=30, tau=0.3, n_iters=4,
                      seeds=np.arange(4, 4 + runs, dtype=np.uint64))
    sim = we.Sim(we.Network(cfg.net), coef, cfg.edges, tau=cfg.tau, m_targ=cfg.m_targ, seeds=cfg.seeds, x0=cfg.x0,
                 max_iters=4, kernel=we.WE_KERNEL_LANE, hist_species=S - 1, hist_lo=0, hist_hi=40,
                 joint_species=joint, joint_bins=bins, joint_width=width)
    sim.step(4)
    got = sim.joint_histogram()
    used = 0
    for r in sorted({0, runs // 2, runs - 1}):
        o = orc.OracleWE(cfg, int(cfg.seeds[r]))
        want, n = np.zeros(bins ** len(joint)), 0
        for _ in range(4):
            o.step(1)
            x, w, _, _ = o.walkers()
            n += len(w)
            cell = sum(np.minimum(x[:, s] // width, bins - 1) * bins ** d for d, s in enumerate(joint))
            want += np.bincount(cell, weights=w, minlength=len(want))
        np.testing.assert_allclose(got[r], want, rtol=n * 2.0 ** -52, atol=0)
        used = max(used, int((want > 0).sum()))
    assert used > 3
