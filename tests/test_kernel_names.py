"""we_propagation_kernel's names: a variant of the lane kernels each, and for the
group kernels the leading template arguments of the kernel that is launched, of
which the library holds every one (the blocks of at most two reactions included)."""
import os
import re

import numpy as np
import pytest

from paper_1303_5986_amd import workloads as wl

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1303_5986_amd", "libwe.so")


def test_group_kernels_of_the_library():
    """Mangled as <L, tables in LDS, block class, descriptor form, register slots>."""
    if not os.path.exists(LIB):
        pytest.skip("libwe.so not built")
    found = set(re.findall(rb"ssa_group_kernelILi(\d+)ELb([01])ELi(\d+)E\d+(RxnDesc2?)Li(\d+)EE", open(LIB, "rb").read()))
    want = {(str(L).encode(), lds, cls, d, slots) for L in (2, 4, 8, 16, 32) for d in (b"RxnDesc", b"RxnDesc2")
            for lds, cls, slots in ((b"1", b"4", b"2"), (b"1", b"4", b"4"), (b"1", b"8", b"8"), (b"1", b"0", b"0"),
                                    (b"0", b"0", b"0"))}
    assert found == want


def _net(S, R, third):
    n = [f"X{i}" for i in range(S)]
    rx = [({n[i % S]: 3}, {n[i % S]: 2}, 0.01) if third and i == 0 else
          ({n[i % S]: 1}, {n[(i + 1) % S]: 1}, 0.5 + 0.1 * i) for i in range(R)]
    return wl.Network.from_reactions(n, rx)


@pytest.mark.gpu
@pytest.mark.parametrize("S,R,third,kernel,wpw,name", [
    (6, 8, False, 1, 0, "ssa_lane_pool_kernel<8,8,true>"), (6, 8, True, 1, 0, "ssa_lane_pool_kernel<8,8>"),
    (6, 9, False, 1, 0, "ssa_lane_pool_kernel<8,16>"), (2, 8, False, 1, 0, "ssa_lane_pool_kernel<2,8>"),
    (6, 16, False, 3, 8, "ssa_group_kernel<8, true, 4>"), (6, 17, False, 3, 8, "ssa_group_kernel<8, true, 4>"),
    (6, 33, False, 3, 8, "ssa_group_kernel<8, true, 8>"), (6, 65, False, 3, 8, "ssa_group_kernel<8, true, 0>")])
def test_names(S, R, third, kernel, wpw, name):
    from paper_1303_5986_amd import we
    print(f"case: name of the kernel for {S} species, {R} reactions", flush=True)
    cfg = wl.WEConfig(name="n", net=_net(S, R, third), x0=np.full(S, 3, np.int32), bin_coef=np.eye(S)[0],
                      edges=wl.uniform_edges(0.0, 9.0, 3), m_targ=4, tau=0.1, n_iters=1, seeds=np.array([1], np.uint64))
    sim = we.sim_from_config(cfg, kernel=kernel, walkers_per_wave=wpw, max_iters=1)
    assert sim.propagation_kernel() == name
