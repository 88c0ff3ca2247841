"""New state rows written by the observation (up to 16 species) and by the gather
(more): chains of 1, 8, 16 and 17 species, few and many runs, with and without
a joint histogram.  Ensembles equal the CPU oracle's bit for bit; the histogram
equals the weights' own sum to n u per entry (it adds in another order)."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _chain(S):
    names = [f"X{i}" for i in range(S)]
    rx = [({names[i]: 1}, {names[i + 1]: 1}, 1.0 + 0.1 * i) for i in range(S - 1)]
    rx += [({}, {names[0]: 1}, 9.0), ({names[-1]: 1}, {}, 0.4)]
    return wl.Network.from_reactions(names, rx)


@pytest.mark.parametrize("S,runs,joint", [(1, 2, False), (8, 3, True), (16, 70, False), (16, 2, True), (17, 2, True),
                                          (17, 66, False)])
def test_rows_and_histogram(S, runs, joint):
    print(f"case: observed rows, {S} species, {runs} runs, joint {joint}", flush=True)
    from paper_1303_5986_amd import we
    coef = np.zeros(S)
    coef[-1] = 1.0
    cfg = wl.WEConfig(name="chain", net=_chain(S), x0=np.full(S, 3, np.int32), bin_coef=coef,
                      edges=wl.uniform_edges(0.0, 30.0, 15), m_targ=9, tau=0.3, n_iters=5,
                      seeds=np.arange(4, 4 + runs, dtype=np.uint64), hist_species=S - 1, hist_lo=0, hist_hi=40)
    if joint:
        cfg.joint_species = [0, S - 1]
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=5, joint=joint)
    ors = {r: orc.OracleWE(cfg, int(cfg.seeds[r])) for r in sorted({0, runs // 2, runs - 1})}
    ref = {r: np.zeros(41) for r in ors}
    for it in range(5):
        sim.step(1)
        for r, o in ors.items():
            o.step(1)
            x, w, b, p = sim.walkers(r)
            for g, e in zip((x, w, b, p), o.walkers()):
                assert np.array_equal(np.asarray(g).view(np.uint8), np.asarray(e).view(np.uint8)), (it, r)
            ok = x[:, S - 1] <= 40
            ref[r] += np.bincount(x[ok, S - 1], weights=w[ok], minlength=41)
    hist, _ = sim.histogram_accum()
    for r in ors:
        np.testing.assert_allclose(hist[r], ref[r], rtol=5 * 135 * 2.0 ** -52, atol=0)
    if joint:
        total = sim.joint_histogram()
        np.testing.assert_allclose(total.sum(axis=1), 5.0, rtol=5 * 135 * 2.0 ** -52)
