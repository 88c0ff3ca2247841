"""As many bins as a grid may have: around the number where the placement's tables
share their LDS (7600), around the one where they would not fit a CU otherwise
(7781), and at the limit of 8192, on one axis and on two, alone and in a batch, with
the weight-equalizing rule and in a replayed graph.  Bit for bit the CPU oracle."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl


def _config(nb, m, rule, two_axes=0):
    base = wl.schlogl_config(n_runs=2, seed0=61, n_iters=6)
    cfg = dataclasses.replace(base, name="bins", m_targ=m, tau=0.1, tgt_thr=130.0, resample_rule=rule,
                              edges=wl.uniform_edges(0.0, 0.25 * nb, nb))
    if two_axes:
        n2 = nb // two_axes
        cfg = dataclasses.replace(cfg, edges=wl.uniform_edges(70.0, 134.0, two_axes), bin_coef2=np.array([1.0]),
                                  edges2=wl.uniform_edges(60.0, 124.0, n2))
    return cfg


def _check(sim, cfg, n, what):
    for r, s in enumerate(cfg.seeds):
        o = orc.OracleWE(cfg, int(s))
        o.step(n)
        for g, e, part in zip(sim.walkers(r), o.walkers(), ("counts", "weights", "bins", "parents")):
            assert np.array_equal(np.asarray(g).view(np.uint8), np.asarray(e).view(np.uint8)), (what, r, part)
        assert np.array_equal(sim.flux(r), o.flux), (what, r)


@pytest.mark.gpu
@pytest.mark.parametrize("nb,m,rule,two_axes", [(7600, 2, 0, 0), (7601, 3, 1, 0), (7781, 2, 0, 0), (7782, 2, 0, 0),
                                                (8192, 1, 0, 0), (8192, 3, 1, 0), (8192, 2, 0, 64)])
def test_sim_and_batch_match_oracle(nb, m, rule, two_axes):
    from paper_1303_5986_amd import we
    print(f"case: {nb} bins x {m}, rule {rule}, {'two axes' if two_axes else 'one axis'}", flush=True)
    cfg = _config(nb, m, rule, two_axes)
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=6)
    sim.step(2)
    sim.graph_capture(2)
    sim.graph_replay(2)
    _check(sim, cfg, 6, "sim")
    b = we.Batch([cfg, wl.birth_death_config()], max_iters=6, kernels=[we.WE_KERNEL_LANE] * 2)
    b.step(6)
    _check(b.members[0], cfg, 6, "batch")
