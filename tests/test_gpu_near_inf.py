"""Near field with one infinite force: the rows whose near lists hold it are infinite
with the sign of their kernel entry, not NaN.

A lane whose share of the sources ends before its wave's longest one must not add its
last source again, not even times zero. Only j's force is not zero, so a row of another
leaf gets K(x_i - x_j) F_j alone where (leaf of i, leaf of j) is in P^H. Every source is
tried, so that it is the last one of many shares.
"""
import numpy as np
import pytest
import torch

import paper_2505_08174_amd as hh
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "bf16", "bf16_split"])
@pytest.mark.parametrize("n,c_leaf", [(900, 16), (1500, 33)])
def test_infinite_force(n, c_leaf, prec):
    from gpu_common import ctx, dev, say
    say("infinite force", n, c_leaf, prec)
    X = wl.lattice_cube(n, 0.1, seed=n)
    Ws, bs = wl.mlp_weights(1)
    hm = hh.HMatrix(ctx(), dev(X), hh.Kernel.mlp(ctx(), (Ws, bs)), c_leaf, 1.0, 1e-4, prec)
    ex = hm.tree.export()
    nodes, perm = ex["nodes"], ex["perm"]
    _, H = hm.part.export()
    leaf = np.empty(n, np.int64)
    for m in np.flatnonzero(nodes[:, 2] < 0):
        leaf[perm[nodes[m, 0]:nodes[m, 1]]] = m
    F = torch.zeros((n, 3), dtype=torch.float32, device="cuda:0")
    for j in range(0, n, 7):
        F[j, 0] = 1.0
        one = (hm @ F).cpu().numpy()
        F[j, 0] = float("inf")
        U = (hm @ F).cpu().numpy()
        F[j] = 0.0
        near = np.isin(leaf, H[H[:, 1] == leaf[j], 0])
        near[j] = False
        want = np.where(one[near] != 0, np.copysign(np.inf, one[near]), np.nan)
        assert np.array_equal(U[near], want, equal_nan=True), (j, np.isnan(U[near]).sum())
