"""Block lists that outgrow the room a partition walk starts with (dense mode, narrow
admissibility): equal to the oracle's, and no level of the walk is run more often than
its lists have to grow.

Levels are launched eight at a time. A list that has to grow is at least doubled, so it
grows at most log2(length / room) times, each of which costs one more batch of launches;
in dense mode the lists of one system are sized beforehand.
"""
import math

import numpy as np
import pytest
import torch

import paper_2505_08174_amd as hh
import workloads as wl
from oracle import partition as OP
from oracle import tree as OT

pytestmark = pytest.mark.gpu


def _launches(fn):
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA, ProfilerActivity.CPU]) as prof:
        r = fn()
        torch.cuda.synchronize()
    return r, sum(e.count for e in prof.key_averages() if "k_level" in e.key)


@pytest.mark.parametrize("n,c_leaf,eta,dense", [(4096, 8, 1.0, True), (700, 2, 1.0, True),
                                                (4000, 3, 0.25, False), (2000, 2, 0.12, False)])
def test_lists_that_grow(n, c_leaf, eta, dense):
    from gpu_common import ctx, dev, say
    say("list growth", n, c_leaf, eta, dense)
    X = wl.lattice_cube(n, 0.1, seed=n)
    ref = OT.build_tree(X, c_leaf)
    t = hh.build_tree(ctx(), dev(X), c_leaf)
    nodes = t.export()["nodes"]
    m, leaves = len(nodes), int(np.sum(nodes[:, 2] < 0))
    p, k = _launches(lambda: hh.partition(ctx(), t, eta, dense_mode=dense))
    g, h = p.export()
    if dense:
        assert g.size == 0 and len(h) == leaves ** 2
        assert np.array_equal(h[:, 0], np.repeat(np.unique(h[:, 0]), leaves))
        assert len(np.unique(h[:, 0].astype(np.int64) * m + h[:, 1])) == len(h)
        grow = 0
    else:
        G, H = OP.build_partition(ref, eta)
        assert np.array_equal(g, np.asarray(G, np.int32).reshape(-1, 2))
        assert np.array_equal(h, np.asarray(H, np.int32).reshape(-1, 2))
        assert len(g) > 160 * m + 1024 or len(h) > 64 * m + 1024
        # a frontier holds no more than all blocks below it: four sons of each parent
        grow = sum(max(0, math.ceil(math.log2(have / room))) for have, room in
                   [(len(g), 160 * m + 1024), (len(h), 64 * m + 1024)] +
                   2 * [(4 * (len(g) + len(h)), 160 * m + 1024)])
    parent = {}
    for i, nd in enumerate(nodes):
        for s in (int(nd[2]), int(nd[3])):
            if s >= 0:
                parent[s] = i
    depth = max(sum(1 for _ in iter(_up(parent, i))) for i in range(m))
    # (k = 0: this profiler sees no kernels)
    assert k <= 8 * (math.ceil((depth + 1) / 8) + grow), (k, depth, grow)


def _up(parent, i):
    while i in parent:
        yield i
        i = parent[i]
