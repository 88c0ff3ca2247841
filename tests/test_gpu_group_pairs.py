"""The group kernel on networks of reactions of at most two molecules
(c x1 (x2 - hom) with an extra species of count 1): species counts on both sides
of a multiple of four, every number of lanes, register blocks of up to four
and eight reactions and longer blocks, and copy numbers from 0 up.  Walkers and
weights equal the oracle's up to the 1% that a sum rounding across a boundary
may change."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,R,wpw", [(3, 8, 32), (4, 16, 16), (7, 40, 8), (8, 63, 8), (13, 130, 4), (31, 250, 2)])
def test_pair_propensities_match_oracle(S, R, wpw):
    from paper_1303_5986_amd import we
    print(f"case: group kernel, pair propensities S={S} R={R} walkers per wave {wpw}", flush=True)
    net = wl.random_network(70 + S, S, R, frac_uni=0.3, rate_lo=1e-2, rate_hi=1.0)
    rng = np.random.default_rng(S)
    x0 = rng.integers(0, 4, size=S).astype(np.int32)
    coef = np.zeros(S)
    coef[0] = 1.0
    cfg = wl.WEConfig(name="pairs", net=net, x0=x0, bin_coef=coef, edges=np.array([0, 1, 2, 4, 8.]), m_targ=6,
                      tau=0.1, n_iters=10, seeds=np.array([3, 4], np.uint64))
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_GROUP, walkers_per_wave=wpw, max_iters=10)
    sim.step(10)
    same = total = 0
    for r in range(2):
        o = orc.OracleWE(cfg, int(cfg.seeds[r]))
        o.step(10)
        x, w, _, _ = sim.walkers(r)
        ox, ow, _, _ = o.walkers()
        assert abs(w.sum() - 1.0) < 1e-12
        if len(w) == len(ow):
            same += int(((x == ox).all(axis=1) & (w == ow)).sum())
        total += len(ow)
    assert same >= 0.99 * total, (same, total)
