"""FP32 near field: a weight keeps every bit of its FP32 value.

The third hidden layer is saturated, so every output is 64 times the one weight w of the
output layer. w' = 1 + 2^-12 fits two FP16 numbers, w = w' + 2^-23 does not (its last bit
is a quarter of their spacing), and 64 w and 64 w' are FP32 numbers: the velocities
of the two networks differ by the factor w / w' up to the roundings that follow (two per
network and entry, each at most 2^-24: 7e-8 together, 2e-9 in the mean of 1,400 entries;
bound 1e-8, and the difference to be seen is 1.2e-7).
"""
import numpy as np
import pytest
import torch

import paper_2505_08174_amd as hh
import workloads as wl

pytestmark = pytest.mark.gpu


def velocities(n, w, inp):
    from gpu_common import ctx, dev
    rng = np.random.default_rng(5)
    Ws = [rng.uniform(-0.5, 0.5, s) for s in [(64, 3), (64, 64), (64, 64)]]
    Ws.append(np.full((9, 64), w))
    bs = [np.zeros(64), np.zeros(64), np.full(64, 100.0), np.zeros(9)]
    kern = hh.Kernel.mlp(ctx(), (Ws, bs), input_mode=inp)
    F = np.zeros((n, 3))
    F[n // 2, 0] = 1.0
    hm = hh.HMatrix(ctx(), dev(wl.lattice_cube(n, 0.1, seed=n)), kern, c_leaf=50, prec="fp32",
                    dense_mode=True)
    U = (hm @ dev(F, torch.float32)).double().cpu().numpy()
    return np.delete(U, n // 2, axis=0)


@pytest.mark.parametrize("inp", ["direction", "displacement"])
def test_last_bit_of_a_weight(inp):
    from gpu_common import say
    say("near weights", inp)
    w1 = 1.0 + 2.0 ** -12
    w = w1 + 2.0 ** -23
    ratio = velocities(471, w, inp) / velocities(471, w1, inp)
    assert abs(ratio.mean() - w / w1) <= 1e-8, ratio.mean() - 1.0
