"""FP32 near field with networks whose rows differ in size.

Layers 2-4 run on FP16 parts under a power of two per row, so rows of very small,
very large and zero weights must keep the FP32 form's accuracy. F has one entry,
so every other row of U is one kernel entry times F (no cancellation between
pairs); rows are compared with the FP64 oracle relative to the largest.

Bound 2e-5: an activation is off by at most a few 2^-23 (1 - 2 / (2^y + 1) and its
split), a pre-activation by that times the row's sum of |W| (below 8 with the
uniform weights here, about 1 with random signs); three layers and the output layer
on top of each other stay below 2e-6, the largest entry is of the order of the
output row's weights, and ten is room for directions in which entries are small.
"""
import math

import numpy as np
import pytest
import torch

import paper_2505_08174_amd as hh
import workloads as wl
from oracle.kernels import MLP, mlp_kernel

pytestmark = pytest.mark.gpu


def network(form, rng):
    Ws, bs = [], []
    for r, c in [(64, 3), (64, 64), (64, 64), (9, 64)]:
        lim = 1.0 / math.sqrt(c)
        Ws.append(rng.uniform(-lim, lim, (r, c)))
        bs.append(rng.uniform(-lim, lim, r))
    if form == "zero rows":
        for i, m in [(1, 5), (2, 40), (3, 4)]:
            Ws[i][m] = 0.0
            bs[i][m] = 0.0
    elif form == "small rows":
        for i in (1, 2):
            f = 10.0 ** rng.uniform(-8, 0, 64)
            Ws[i] *= f[:, None]
            bs[i] *= f
    elif form == "tiny":
        Ws[1] *= 1e-40
        bs[1] *= 0.0
        Ws[3] *= 1e-25
        bs[3] *= 1e-25
    elif form == "huge":
        bs[2][:8] = np.where(np.arange(8) % 2, 1e35, -1e35)
        Ws[3] *= 1e30
        bs[3] *= 1e30
    return Ws, bs


@pytest.mark.parametrize("inp", ["direction", "displacement"])
@pytest.mark.parametrize("form", ["plain", "zero rows", "small rows", "tiny", "huge"])
@pytest.mark.parametrize("n", [40, 161])
def test_single_entries(n, form, inp):
    from gpu_common import ctx, dev, say
    say("near x2", n, form, inp)
    Ws, bs = network(form, np.random.default_rng(3))
    kern = hh.Kernel.mlp(ctx(), (Ws, bs), input_mode=inp)
    X = wl.lattice_cube(n, 0.1, seed=n)
    F = np.zeros((n, 3))
    j = n // 3
    F[j] = [0.5, -1.0, 0.25]
    hm = hh.HMatrix(ctx(), dev(X), kern, c_leaf=33, prec="fp32", dense_mode=True)
    U = (hm @ dev(F, torch.float32)).double().cpu().numpy()
    others = np.arange(n) != j
    ref = mlp_kernel(X[others] - X[j], MLP(Ws, bs), inp) @ F[j]
    row = np.max(np.linalg.norm(U[others] - ref, axis=1)) / np.max(np.linalg.norm(ref, axis=1))
    assert row <= 2e-5, row
