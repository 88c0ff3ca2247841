"""The LDS bytes that bench.py counts per event of the factored-table wave kernel, by
hand, in the kernel's two forms."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
from paper_1303_5986_amd import workloads as wl  # noqa: E402


def test_pair_form():
    """A + B -> C and C -> 0: A and B each in one reaction's reactants, C in one.
    Dependents 3 and 1, mean 2; changed species 3 and 1, mean 2.  A dependent
    moves its 4-byte entry, 8-byte constant, one 4-byte count and a 16-byte add."""
    net = wl.Network.from_reactions(["A", "B", "C"], [({"A": 1, "B": 1}, {"C": 1}, 1.0), ({"C": 1}, {}, 1.0)])
    assert bench.lds_bytes_per_event_fact(net) == 64 * 32 + 2 * 12 + 2 * (16 + 16) + 512


def test_general_form():
    """3 A -> B and B -> A: dependents 2 and 2, changed species 2; a dependent moves
    its 2-byte id, 16-byte descriptor and four 4-byte counts."""
    net = wl.Network.from_reactions(["A", "B"], [({"A": 3}, {"B": 1}, 1.0), ({"B": 1}, {"A": 1}, 1.0)])
    assert bench.lds_bytes_per_event_fact(net) == 64 * 32 + 2 * 12 + 2 * (34 + 16) + 512
