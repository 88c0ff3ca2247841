"""Merges in rounds under the weight-equalizing rule, with targets of at most
128: bins around a wave's 64 lanes, around the sizes where the rounds start
and end, and with few and many merges; weights that tie, that are zero, and that
span many decades.  Bit for bit the oracle's ensembles, under both rules, alone
and in a batch."""
import numpy as np
import pytest

from oracle import oracle as orc
from test_gpu_resample_big import KINDS, _check, _config

pytestmark = pytest.mark.gpu

COUNTS = [1, 7, 8, 9, 19, 20, 21, 63, 64, 65, 66, 76, 77, 99, 101, 113, 127, 128, 129, 130, 200, 255, 256, 257, 300]


@pytest.mark.parametrize("rule,kind", [(r, k) for r in (0, 1) for k in KINDS if (r, k) != (1, "tiny")])
@pytest.mark.parametrize("m", [8, 64, 100])
def test_rounds(m, rule, kind):
    from paper_1303_5986_amd import we
    print(f"case: merges in rounds, bins x {m}, {kind}, rule {rule}", flush=True)
    rng = np.random.default_rng(100 * m + KINDS.index(kind))
    cfg, x, w = _config(rng, 400, m, COUNTS, kind, rule)
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=2)
    sim.set_ensemble(0, x, w)
    o = orc.OracleWE(cfg, 77, init_x=x, init_w=w)
    for it in range(2):
        sim.step(1)
        o.step(1)
        _check(sim.walkers(0), o, it)
    b = we.Batch([cfg], max_iters=2, kernels=[we.WE_KERNEL_LANE])
    b.members[0].set_ensemble(0, x, w)
    b.step(1)
    o = orc.OracleWE(cfg, 77, init_x=x, init_w=w)
    o.step(1)
    _check(b.members[0].walkers(0), o, 0)
