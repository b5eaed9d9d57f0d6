"""Sorting, scans and the partition walk at the edges of their one-workgroup and
tiled forms: trees and block lists equal to the oracle's, bit for bit.

The Morton sort has n elements and the node, P^G and P^H sorts as many as the
lists below, so the sizes put each of them below, at and above the 8,192 pairs
of the one-workgroup sort and the 16,384 values of the one-workgroup scan; tiny
leaves make lists far longer than the room a walk starts with.
"""
import numpy as np
import pytest

import paper_2505_08174_amd as hh
import workloads as wl
from oracle import partition as OP
from oracle import tree as OT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c_leaf,eta", [(1, 2, 1.0), (2, 2, 1.0), (1023, 2, 1.0),
                                          (1025, 16, 0.3), (4000, 3, 0.25), (8191, 64, 1.0),
                                          (8192, 64, 1.0), (8193, 64, 1.0), (20000, 33, 1.0)])
def test_tree_and_lists_match_oracle(n, c_leaf, eta):
    from gpu_common import ctx, dev, say
    say("lists", n, c_leaf, eta)
    X = wl.lattice_cube(n, 0.1, seed=n)
    tr = OT.build_tree(X, c_leaf)
    t = hh.build_tree(ctx(), dev(X), c_leaf)
    ex = t.export()
    assert np.array_equal(ex["perm"], tr.perm)
    assert np.array_equal(ex["nodes"], tr.nodes)
    assert np.array_equal(ex["bbox"], tr.bbox)
    G, H = OP.build_partition(tr, eta)
    g, h = hh.partition(ctx(), t, eta).export()
    assert np.array_equal(g, np.asarray(G, np.int32).reshape(-1, 2))
    assert np.array_equal(h, np.asarray(H, np.int32).reshape(-1, 2))

