"""Split and merge of large bins: merges in rounds (bins of 257 to 2048
walkers above M, with M above 128), hand-outs of many copies at once, the
bin-parallel launch with more than 32 bins, and the batched one.  Weights that
tie (equal, dyadic, zero), that span many decades, that repeat in groups and
that are subnormal; every bin of a run another size.  Bit for bit the oracle's
ensembles, under both rules."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl

pytestmark = pytest.mark.gpu

KINDS = ["equal", "dyadic", "zeros", "uniform", "decades", "groups", "tiny"]


def _weights(rng, n, kind):
    return {"equal": lambda: np.full(n, 1.0 / 64), "dyadic": lambda: 2.0 ** -rng.integers(3, 9, n).astype(float),
            "zeros": lambda: rng.choice([0.0, 1 / 32.0, 1 / 128.0], n), "uniform": lambda: rng.uniform(0, 1, n) / n,
            "decades": lambda: 10.0 ** rng.uniform(-25, 0, n), "groups": lambda: rng.choice(rng.uniform(0, 1, 5), n),
            "tiny": lambda: 5e-324 * rng.integers(0, 40, n)}[kind]()


def _config(rng, n_bins, m, counts, kind, rule):
    net = wl.Network.from_reactions(["X", "Y"], [({"X": 1}, {"X": 1, "Y": 1}, 0.0)])
    cfg = wl.WEConfig(name="frozen", net=net, x0=np.array([0, 0], np.int32), bin_coef=np.array([1.0, 0.0]),
                      edges=wl.uniform_edges(0.0, float(n_bins), n_bins), m_targ=m, tau=1.0, n_iters=2,
                      seeds=np.array([77], np.uint64), resample_rule=rule)
    b = np.repeat(np.arange(len(counts)), counts)
    x = np.stack([b, rng.integers(0, 50, len(b))], axis=1).astype(np.int32)
    w = np.concatenate([_weights(rng, c, kind) for c in counts])
    perm = rng.permutation(len(b))
    return cfg, x[perm], w[perm]


def _check(got, o, it):
    for a, c in zip(got, o.walkers()):
        assert len(a) == len(c) and np.array_equal(a, c), it


# not ("tiny", 1): the ideal weight of a bin of subnormal weights rounds to 0, and
# a walker's needed copies are then infinity as an integer, which C leaves
# undefined (the oracle and the GPU convert it to different ends of the range)
@pytest.mark.parametrize("kind,rule", [(k, 0) for k in KINDS] + [(k, 1) for k in KINDS if k != "tiny"])
def test_bin_parallel(kind, rule):
    from paper_1303_5986_amd import we
    print(f"case: large bins, one run of 40 bins x 160, {kind}, rule {rule}", flush=True)
    rng = np.random.default_rng(KINDS.index(kind))
    counts = [1, 2, 3, 63, 64, 65, 127, 128, 129, 159, 160, 161, 255, 256, 257, 511, 512, 513, 700, 1023, 1]
    cfg, x, w = _config(rng, 40, 160, counts, kind, rule)
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=2)
    sim.set_ensemble(0, x, w)
    o = orc.OracleWE(cfg, 77, init_x=x, init_w=w)
    for it in range(2):
        sim.step(1)
        o.step(1)
        _check(sim.walkers(0), o, it)


@pytest.mark.parametrize("m,counts", [(512, [513, 2047, 2048, 2049, 1, 300, 500, 100]), (129, [130, 900, 0, 2]),
                                      (5, [6, 30, 1, 2]), (700, [1401, 64, 699, 701])])
def test_one_workgroup_and_batch(m, counts):
    """Few bins: split and merged by the run's workgroup on its own sim; one
    wave per bin in a batch, whose member runs on from a first iteration."""
    from paper_1303_5986_amd import we
    print(f"case: large bins, {len(counts)} bins x {m}", flush=True)
    rng = np.random.default_rng(m)
    cfg, x, w = _config(rng, max(len(counts), 16), m, counts, "decades", 0)
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=2)
    sim.set_ensemble(0, x, w)
    o = orc.OracleWE(cfg, 77, init_x=x, init_w=w)
    sim.step(1)
    o.step(1)
    _check(sim.walkers(0), o, 0)
    # a network that moves: each interval's bins gain and lose many walkers
    mv = dataclasses.replace(wl.birth_death_config(), m_targ=m, edges=wl.uniform_edges(30.0, 50.0, 10), tau=2.0,
                             seeds=np.array([m], np.uint64))
    b = we.Batch([mv, dataclasses.replace(mv, resample_rule=1), cfg], max_iters=6, kernels=[we.WE_KERNEL_LANE] * 3)
    b.step(6)
    b.synchronize()
    for i, c in enumerate((mv, dataclasses.replace(mv, resample_rule=1))):
        o = orc.OracleWE(c, m)
        o.step(6)
        _check(b.members[i].walkers(0), o, i)
