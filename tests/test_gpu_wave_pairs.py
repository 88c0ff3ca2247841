"""The wave kernels on networks of reactions of at most two molecules, whose
propensities are formed as c x1 (x2 - hom) with an extra species of count 1
for an absent reactant: species counts on both sides of a multiple of four
(the extra count's place in the walker's LDS slice), up to the factored
format's 512 species and past it (the descriptor tables), and copy numbers from
0 up, where a pair of equal molecules has none or one combination.  Walkers and
weights equal the oracle's; as on every wave path, 1% may differ (an event
changes when a sum rounds across a boundary)."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,R,kernel", [(7, 40, "fact"), (8, 60, "fact"), (9, 64, "fact"), (511, 600, "fact"),
                                        (512, 600, "fact"), (513, 600, "lds")])
def test_pair_propensities_match_oracle(S, R, kernel):
    from paper_1303_5986_amd import we
    print(f"case: wave kernels, pair propensities S={S} R={R}", flush=True)
    net = wl.random_network(90 + S, S, R, frac_uni=0.3, rate_lo=1e-2, rate_hi=1.0)
    rng = np.random.default_rng(S)
    x0 = rng.integers(0, 4, size=S).astype(np.int32)
    coef = np.zeros(S)
    coef[0] = 1.0
    cfg = wl.WEConfig(name="pairs", net=net, x0=x0, bin_coef=coef, edges=np.array([0, 1, 2, 4, 8.]), m_targ=6,
                      tau=0.1, n_iters=10, seeds=np.array([3, 4], np.uint64))
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_WAVE, max_iters=10)
    assert kernel in sim.propagation_kernel()
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
