"""Split and merge with targets above 128 where many bins share the chip: every
room for merges in rounds (512, 1024 and 2048 walkers, none) at the edges of the
rule that picks it (512 waves, targets of 384 and 768, both rules), with bins
below, at and above the room and the registers' 512.  Frozen ensembles of random
weights, the same for the sim and the batch; bit for bit the CPU oracle."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1303_5986_amd import workloads as wl
from test_gpu_resample_big import _config

pytestmark = pytest.mark.gpu

COUNTS = [1, 64, 65, 129, 200, 256, 257, 383, 384, 385, 511, 512, 513, 600, 769, 1023, 1024, 1025]


@pytest.mark.parametrize("rule", [0, 1])
@pytest.mark.parametrize("m,runs", [(129, 12), (129, 13), (384, 13), (385, 13), (768, 13), (769, 13)])
def test_room_for_merges(m, runs, rule):
    """40 bins: 12 runs are 480 waves, 13 are 520."""
    from paper_1303_5986_amd import we
    print(f"case: {runs} runs of 40 bins x {m}, rule {rule}", flush=True)
    counts = [c for c in COUNTS if m > 200 or c not in (200, 769, 1023, 1024)]   # within 40 m slots
    ens = {}
    for r, kind in ((0, "decades"), (7, "dyadic"), (runs - 1, "groups")):
        rng = np.random.default_rng(r + m)
        cfg, x, w = _config(rng, 40, m, list(rng.permutation(counts)), kind, rule)
        ens[r] = (x, w)
    seeds = np.full(runs, 77, np.uint64)
    sim = we.sim_from_config(cfg.with_seeds(seeds), kernel=we.WE_KERNEL_LANE, max_iters=2)
    b = we.Batch([wl.birth_death_config(), cfg.with_seeds(seeds)], max_iters=2, kernels=[we.WE_KERNEL_LANE] * 2)
    for r, (x, w) in ens.items():
        sim.set_ensemble(r, x, w)
        b.members[1].set_ensemble(r, x, w)
    sim.step(2)
    b.step(2)
    for r, (x, w) in ens.items():
        o = orc.OracleWE(cfg, 77, init_x=x, init_w=w)
        o.step(2)
        for got in (sim.walkers(r), b.members[1].walkers(r)):
            for g, e in zip(got, o.walkers()):
                assert len(g) == len(e) and np.array_equal(g, e), r
