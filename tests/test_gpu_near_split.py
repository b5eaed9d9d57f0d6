"""Near field at the edges of its 64-target waves and of its source shares.

In dense mode every pair is a near pair, so the product is the dense sum: the
sizes below sit around one wave of targets, make the shares of the sources
shorter than one source and the leaves (and so the near lists' entries) odd,
even and single. Bounds as for the dense-mode products: FP64 1e-10 (rounding
of N-term sums); FP32 1e-5 (a few 1e-7 per entry, times sum|K F| / |sum K F|
below ~10); BF16 hi + lo 1e-4 (about 1e-6 per entry times that ratio, with
room for the few-term sums of the smallest systems); BF16 5e-3 (1e-4 per
entry, likewise).
"""
import numpy as np
import pytest
import torch

import paper_2505_08174_amd as hh
import workloads as wl
from oracle import dense as OD

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-5, "bf16_split": 1e-4, "bf16": 5e-3}


@pytest.mark.parametrize("n,c_leaf", [(1, 2), (2, 2), (5, 2), (63, 7), (64, 16), (65, 9),
                                      (129, 33), (700, 64), (1025, 16)])
@pytest.mark.parametrize("kind,prec", [("rpy", "fp64"), ("rpy", "fp32"), ("mlp", "fp32"),
                                       ("mlp", "bf16_split"), ("mlp", "bf16")])
def test_dense_product_at_edge_sizes(kind, prec, n, c_leaf):
    from gpu_common import ctx, dev, kernels, say
    say("near split", kind, prec, n, c_leaf)
    X = wl.lattice_cube(n, 0.1, seed=n)
    F = wl.normal_forces(n, seed=n)
    ko, kg = kernels(kind)
    ref = OD.dense_u(X, F, ko)
    hm = hh.HMatrix(ctx(), dev(X), kg, c_leaf=c_leaf, prec=prec, dense_mode=True)
    U = (hm @ dev(F, torch.float64 if prec == "fp64" else torch.float32)).double().cpu().numpy()
    row = np.max(np.linalg.norm(U - ref, axis=1)) / np.max(np.linalg.norm(ref, axis=1))
    assert row <= TOL[prec], (row, TOL[prec])
