"""Weights that are not finite (only a checkpoint can bring them in from outside):
bins of 1 to 700 walkers, all of them or some of them not a number or infinite, in
every way a run is resampled -- by its workgroup with the arrays in LDS and in device
memory, by bin, in registers, in rounds -- under both rules.  The next interval ends
and latches a device fault, which every read reports."""
import numpy as np
import pytest

from test_gpu_resample_big import _config

pytestmark = pytest.mark.gpu


def _patched(path, w, bad, value):
    """The checkpoint's weights w (as bytes) with the entries `bad` replaced."""
    data = open(path, "rb").read()
    at = data.find(w.tobytes())
    assert at > 0 and data.find(w.tobytes(), at + 1) < 0
    v = w.copy()
    v[bad] = value
    open(path, "wb").write(data[:at] + v.tobytes() + data[at + 8 * len(w):])


@pytest.mark.parametrize("bins,m", [(4, 64), (4, 700), (40, 64), (40, 160), (12, 1200)])
@pytest.mark.parametrize("rule", [0, 1])
@pytest.mark.parametrize("value,share", [(np.nan, 1.0), (np.nan, 0.5), (np.inf, 1.0), (np.inf, 0.3)])
def test_fault_is_latched(tmp_path, bins, m, rule, value, share):
    from paper_1303_5986_amd import we
    print(f"case: {value} in {share} of the weights, {bins} bins x {m}, rule {rule}", flush=True)
    rng = np.random.default_rng(bins * m + rule)
    counts = [c for c in (64, 1, 63, 65, 128, 200, 256, 300, 700) if c <= 2 * m][:bins]
    cfg, x, w = _config(rng, bins, m, counts, "uniform", rule)
    net = we.Network(cfg.net)
    sim = we.sim_from_config(cfg, kernel=we.WE_KERNEL_LANE, max_iters=3, network=net)
    sim.set_ensemble(0, x, w)
    path = str(tmp_path / "c.ck")
    sim.save(path)
    sim.close()
    _patched(path, w, rng.random(len(w)) < share, value)
    sim = we.Sim.load(net, path)
    assert len(sim.walkers(0)[1]) == len(w)
    sim.step(2)
    for read in (sim.synchronize, lambda: sim.walkers(0), lambda: sim.flux(0, 0, 1)):
        with pytest.raises(we.WEError, match="weight"):
            read()
