"""Batches of very different members: many runs of few bins beside one run of many
bins and a crowd of small ones, with targets on both sides of 128.  Every member
equals the same run stepped on its own, and the batch costs about what its members
cost."""
import dataclasses
import time

import numpy as np
import pytest

from paper_1303_5986_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _bd(runs, bins, m, rule=0, seed=1):
    c = wl.birth_death_config(n_runs=runs, seed0=seed)
    return dataclasses.replace(c, edges=wl.uniform_edges(0.0, 100.0, bins), m_targ=m, tau=1.0, resample_rule=rule)


@pytest.mark.parametrize("m,rule", [(8, 0), (20, 1), (130, 0), (130, 1)])
def test_members_equal_standalone(m, rule):
    from paper_1303_5986_amd import we
    print(f"case: uneven batch, targets of {m}, rule {rule}", flush=True)
    cfgs = [_bd(520, 9, m, rule), _bd(1, 2500, 3, rule, 2), _bd(3, 33, m, rule, 5)] + [_bd(1, 20, 4, seed=i) for i in range(20)]
    b = we.Batch(cfgs, max_iters=6, kernels=[we.WE_KERNEL_LANE] * len(cfgs))
    b.step(2)
    b.graph_capture(2)
    b.graph_replay(2)
    b.synchronize()
    for cfg, mem in zip(cfgs[:5], b.members):
        s = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=6)
        s.step(6)
        for r in sorted({0, s.n_runs // 2, s.n_runs - 1}):
            for g, e in zip(mem.walkers(r), s.walkers(r)):
                assert np.array_equal(g, e), (cfg.edges.size, r)


def test_cost_is_the_members_cost():
    """A step of the whole batch takes no longer than three times the steps of its
    parts batched by themselves (measured 1.3 times)."""
    from paper_1303_5986_amd import we
    print("case: uneven batch, time of a step", flush=True)
    many, wide, small = [_bd(512, 16, 8)], [_bd(1, 4000, 1)], [_bd(1, 20, 4, seed=i) for i in range(30)]

    def step_us(cfgs):
        b = we.Batch(cfgs, max_iters=200, kernels=[we.WE_KERNEL_LANE] * len(cfgs))
        b.step(20)
        b.members[0].synchronize()
        best = 1e9
        for _ in range(5):
            t0 = time.perf_counter()
            b.step(20)
            b.members[0].synchronize()
            best = min(best, time.perf_counter() - t0)
        return best / 20 * 1e6

    parts = [step_us(c) for c in (many, wide, small)]
    whole = step_us(many + wide + small)
    print(f"   parts {parts}, whole {whole} us a step", flush=True)
    assert whole < 3 * sum(parts)
