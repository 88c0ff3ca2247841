"""Reading results back: ensembles whose bytes end just before, at and after the
pinned memory's first size (64 KiB), one half (1 MiB) and several halves, only
some of the arrays, histograms of several halves, and several threads at once.
An ensemble set by the caller must come back bit for bit, and so must the
histogram of its first interval against the walkers' own weights (which add up
in another order: rtol n u for n walkers)."""
import ctypes as C
import dataclasses
import threading

import numpy as np
import pytest

from paper_1303_5986_amd import workloads as wl

pytestmark = pytest.mark.gpu

# 20 bytes a walker (one species) and 16 of header
EDGES = [1, 3275, 3276, 3277, 6550, 52427, 52428, 52429, 104858, 200000]


def _sim(n, runs=1):
    from paper_1303_5986_amd import we
    base = wl.birth_death_config(n_runs=runs, seed0=3)
    cfg = dataclasses.replace(base, m_targ=max(1, n // 40 + 1), edges=wl.uniform_edges(0.0, 120.0, 40))
    return we, we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=2)


@pytest.mark.parametrize("n", EDGES)
def test_ensemble_comes_back(n):
    print(f"case: readback of {n} walkers", flush=True)
    we, sim = _sim(n)
    rng = np.random.default_rng(n)
    x = rng.integers(0, 100, (n, 1)).astype(np.int32)
    w = rng.random(n)
    sim.set_ensemble(0, x, w)
    gx, gw, gb, go = sim.walkers(0)
    assert np.array_equal(gx, x) and np.array_equal(gw, w) and len(gb) == n and len(go) == n
    only = np.zeros(sim.cap, np.int32)
    got = C.c_int32(0)
    assert we.load_library().we_get_walkers(sim.handle, 0, C.byref(got), only.ctypes.data_as(C.c_void_p), None, None,
                                            None) == 0
    assert got.value == n and np.array_equal(only[:n], x[:, 0]) and not only[n:].any()


def test_histogram_of_several_halves():
    print("case: readback of a 2.6 MB histogram", flush=True)
    from paper_1303_5986_amd import we
    base = wl.schlogl_config(n_runs=400, seed0=1, n_iters=1)
    cfg = dataclasses.replace(base, recycle=False)
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=1)
    sim.step(1)
    hist, n = sim.histogram_accum()
    assert n == 1
    for r in (0, 131, 262, 399):
        x, w, _, _ = sim.walkers(r)
        ok = (x[:, 0] >= cfg.hist_lo) & (x[:, 0] <= cfg.hist_hi)
        ref = np.bincount(x[ok, 0] - cfg.hist_lo, weights=w[ok], minlength=hist.shape[1])
        np.testing.assert_allclose(hist[r], ref, rtol=len(w) * 2.0 ** -52, atol=0)


def test_threads_read_at_once():
    print("case: readback from four threads", flush=True)
    we, sim = _sim(60000, runs=4)
    rng = np.random.default_rng(1)
    sent = [(rng.integers(0, 100, (n, 1)).astype(np.int32), rng.random(n)) for n in (60000, 10, 30000, 3000)]
    for r, (x, w) in enumerate(sent):
        sim.set_ensemble(r, x, w)
    bad = []

    def read(r):
        for _ in range(5):
            gx, gw, _, _ = sim.walkers(r)
            if not (np.array_equal(gx, sent[r][0]) and np.array_equal(gw, sent[r][1])):
                bad.append(r)

    threads = [threading.Thread(target=read, args=(r,)) for r in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
