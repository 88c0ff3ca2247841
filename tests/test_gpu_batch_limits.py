"""Batches at the limits of a CU: wave members whose reaction tables and counts
would fill the 160 KB of LDS to the last byte (the kernel keeps a word of its own
beside them), and the most species a batch takes.  Members equal the same run
stepped on its own, bit for bit."""
import numpy as np
import pytest

from paper_1303_5986_amd import workloads as wl


def _net(S, R):
    """A decay per species, then conversions along the chain of species."""
    n = [f"X{i}" for i in range(S)]
    rx = [({n[i]: 1}, {}, 0.4 + 0.1 * (i % 7)) for i in range(min(S, R))]
    while len(rx) < R:
        i, step = len(rx) % S, 1 + len(rx) // S
        rx.append(({n[i]: 1}, {n[(i + step) % S]: 1}, 0.3 + 0.05 * (i % 5)))
    return wl.Network.from_reactions(n, rx)


def _config(S, R):
    coef = np.zeros(S)
    coef[0] = 1.0
    return wl.WEConfig(name="limit", net=_net(S, R), x0=np.full(S, 2, np.int32), bin_coef=coef,
                       edges=wl.uniform_edges(0.0, 4.0, 4), m_targ=5, tau=0.002, n_iters=4, seeds=np.array([9], np.uint64))


@pytest.mark.gpu
@pytest.mark.parametrize("S,R", [(3148, 3680), (3151, 3680), (2940, 4096), (3964, 4096)])
def test_tables_that_fill_the_lds(S, R):
    from paper_1303_5986_amd import we
    print(f"case: batched wave kernel, {S} species, {R} reactions", flush=True)
    cfg = _config(S, R)
    b = we.Batch([cfg], max_iters=4, kernels=[we.WE_KERNEL_WAVE])
    b.step(4)
    s = we.sim_from_config(cfg, kernel=we.WE_KERNEL_WAVE, max_iters=4)
    s.step(4)
    assert s.counters()[0] > 0
    for g, e in zip(b.members[0].walkers(0), s.walkers(0)):
        assert np.array_equal(g, e)


@pytest.mark.gpu
@pytest.mark.parametrize("S,fits", [(3968, True), (3969, False)])
def test_most_species(S, fits):
    from paper_1303_5986_amd import we
    print(f"case: batch of {S} species", flush=True)
    cfg = _config(S, 40)
    if fits:
        b = we.Batch([cfg], max_iters=2, kernels=[we.WE_KERNEL_WAVE])
        b.step(2)
        b.synchronize()
    else:
        with pytest.raises(we.WEError):
            we.Batch([cfg], max_iters=2, kernels=[we.WE_KERNEL_WAVE])
