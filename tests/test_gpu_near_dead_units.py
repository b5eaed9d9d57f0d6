"""FP32 near field with units that are zero whatever the input (zero weights and bias):
their weights in the next layer, however large, take no accuracy from the others.

Rows of weights share a power of two in the FP16 parts; a weight of 1e9 on a dead unit
would leave the others of its row (of order 0.1) some 7 of their bits. F has one entry,
so the rows of U are single kernel entries; bound 2e-5 of the largest as for other
networks of FP32 accuracy (a few 2^-23 through four layers of row sums below 8).
"""
import math

import numpy as np
import pytest
import torch

import paper_2505_08174_amd as hh
import workloads as wl
from oracle.kernels import MLP, mlp_kernel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inp", ["direction", "displacement"])
@pytest.mark.parametrize("dead", [1, 2, 3, "chain"])
def test_dead_units(dead, inp):
    from gpu_common import ctx, dev, say
    say("dead units", dead, inp)
    rng = np.random.default_rng(4)
    Ws, bs = [], []
    for r, c in [(64, 3), (64, 64), (64, 64), (9, 64)]:
        lim = 1.0 / math.sqrt(c)
        Ws.append(rng.uniform(-lim, lim, (r, c)))
        bs.append(rng.uniform(-lim, lim, r))
    units = [3, 17, 40]
    first = 1 if dead == "chain" else dead
    Ws[first - 1][units] = 0.0
    bs[first - 1][units] = 0.0
    Ws[first][:, units] = 1e9
    if dead == "chain":   # units that see dead ones only
        only = np.zeros(64, bool)
        only[units] = True
        Ws[1][5, ~only] = 0.0
        bs[1][5] = 0.0
        Ws[2][:, 5] = -1e9
    kern = hh.Kernel.mlp(ctx(), (Ws, bs), input_mode=inp)
    n, j = 161, 50
    X = wl.lattice_cube(n, 0.1, seed=n)
    F = np.zeros((n, 3))
    F[j] = [0.5, -1.0, 0.25]
    hm = hh.HMatrix(ctx(), dev(X), kern, c_leaf=33, prec="fp32", dense_mode=True)
    U = (hm @ dev(F, torch.float32)).double().cpu().numpy()
    others = np.arange(n) != j
    ref = mlp_kernel(X[others] - X[j], MLP(Ws, bs), inp) @ F[j]
    row = np.max(np.linalg.norm(U[others] - ref, axis=1)) / np.max(np.linalg.norm(ref, axis=1))
    assert row <= 2e-5, row
