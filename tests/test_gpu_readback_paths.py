"""Reading results where pinned memory is refused (plain copies), and a device
fault latched before a result of several halves."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_1303_5986_amd import workloads as wl

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

REFUSE = """
int refused;
int hipHostMalloc(void **p, unsigned long n, unsigned f) { (void)n; (void)f; *p = 0; ++refused; return 2; }
"""

CHILD = """
import ctypes, sys
import numpy as np
refuse = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path[:0] = [sys.argv[2], sys.argv[3]]
import dataclasses
from paper_1303_5986_amd import we, workloads as wl
from oracle import oracle as orc
cfg = dataclasses.replace(wl.schlogl_config(n_runs=3, seed0=3, n_iters=6), m_targ=20)
sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=6)
sim.step(6)
for r in range(3):
    o = orc.OracleWE(cfg, int(cfg.seeds[r]))
    o.step(6)
    for g, e in zip(sim.walkers(r), o.walkers()):
        assert len(g) == len(e) and np.array_equal(g, e), r
    assert np.array_equal(sim.flux(r), o.flux)
    n = ctypes.c_int32(0)
    w = np.zeros(sim.cap)
    assert we.load_library().we_get_walkers(sim.handle, r, ctypes.byref(n), None, w.ctypes.data_as(ctypes.c_void_p),
                                            None, None) == 0
    assert np.array_equal(w[:n.value], o.walkers()[1]) and not w[n.value:].any()
hist, n = sim.histogram_accum()
assert n == 6 and abs(hist.sum() - 18.0) < 1e-9
calls = ctypes.c_int.in_dll(refuse, "refused").value
print("refused", calls, flush=True)
assert calls > 0
"""


@pytest.mark.gpu
def test_without_pinned_memory(tmp_path):
    """A process in which hipHostMalloc fails for the library."""
    print("case: readback without pinned memory", flush=True)
    src, so = tmp_path / "refuse.c", tmp_path / "refuse.so"
    src.write_text(REFUSE)
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-o", str(so), str(src)])
    r = subprocess.run([sys.executable, "-c", CHILD, str(so), ROOT, HERE], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.gpu
def test_fault_before_a_result_of_several_halves():
    """A count past its limit: every read says so, however long its result, and
    leaves the caller's array alone."""
    print("case: latched overflow, 3 MB of histograms", flush=True)
    from paper_1303_5986_amd import we
    net = wl.Network.from_reactions(["X"], [({}, {"X": 1}, 50.0)])
    cfg = wl.WEConfig(name="over", net=net, x0=np.array([131000], np.int32), bin_coef=np.array([1.0]),
                      edges=wl.uniform_edges(0.0, 1.0, 4), m_targ=4, tau=10.0, n_iters=2,
                      seeds=np.arange(1, 41, dtype=np.uint64), hist_species=0, hist_lo=0, hist_hi=9999)
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=2)
    sim.step(1)
    L = we.load_library()
    out = np.full(40 * 10000, 7.0)
    n = ctypes.c_int32(-1)
    for _ in range(2):
        assert L.we_histogram_accum(sim.handle, out.ctypes.data_as(ctypes.c_void_p), ctypes.byref(n)) == -5
        assert (out == 7.0).all() and n.value == -1
        with pytest.raises(we.WEError):
            sim.walkers(0)
