"""Batched propagation by chunks of slots: every kernel variant (lane; group
with 2 to 32 lanes, in registers, in LDS and through the cache; wave in both
forms of descriptors), slot counts that no round of a workgroup divides, one
member and many, eager steps and a replayed graph.  Every member equals the
same run stepped on its own, bit for bit."""
import numpy as np
import pytest

from paper_1303_5986_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _random(S, R, runs, bins, m, tau=0.02):
    net = wl.random_network(300 + S + R, S, R, rate_lo=1e-2, rate_hi=1.0)
    x0 = np.random.default_rng(S + R).integers(0, 12, size=S).astype(np.int32)
    coef = np.zeros(S)
    coef[int(np.argmax(x0))] = 1.0
    return wl.WEConfig(name=f"r{S}_{R}", net=net, x0=x0, bin_coef=coef, edges=wl.uniform_edges(0.0, 16.0, bins),
                       m_targ=m, tau=tau, n_iters=0, seeds=np.arange(1, runs + 1, dtype=np.uint64))


LANE, WAVE, GROUP = 1, 2, 3
CASES = {
    "one_wave_member": [((13, 130, 1, 5, 13), WAVE)],
    "group_lanes": [((8, 63, 2, 4, 7), (GROUP, w)) for w in (32, 16, 8, 4, 2)] +
                   [((30, 200, 1, 3, 33), (GROUP, w)) for w in (32, 16, 8, 4, 2)],
    "group_tables_through_cache": [((289, 3000, 1, 3, 9), (GROUP, 2)), ((30, 250, 1, 3, 9), (GROUP, 2))],
    "mixed": [("schlogl", LANE), ("schlogl", WAVE), ((3, 8, 3, 7, 5), LANE), ((5, 16, 2, 3, 41), LANE),
              ((12, 30, 1, 5, 19), LANE), ((8, 63, 1, 1, 1), (GROUP, 8)), ((60, 500, 2, 4, 67), WAVE),
              ((354, 3680, 1, 3, 5), WAVE)],
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_members_equal_standalone(name):
    from paper_1303_5986_amd import we
    print(f"case: batch chunks {name}", flush=True)
    cfgs = [wl.schlogl_config(n_runs=2, seed0=5) if c == "schlogl" else _random(*c) for c, _ in CASES[name]]
    kernels = [k for _, k in CASES[name]]
    b = we.Batch(cfgs, max_iters=20, kernels=kernels)
    b.step(4)
    b.graph_capture(2)
    b.graph_replay(3)
    b.step(2)
    b.synchronize()
    for cfg, kern, m in zip(cfgs, kernels, b.members):
        k, wpw = kern if isinstance(kern, tuple) else (kern, 0)
        s = we.sim_from_config(cfg, kernel=k, walkers_per_wave=wpw, max_iters=20)
        s.step(12)
        for r in range(s.n_runs):
            for a, c in zip(m.walkers(r), s.walkers(r)):
                assert np.array_equal(a, c), (cfg.name, kern, r)
