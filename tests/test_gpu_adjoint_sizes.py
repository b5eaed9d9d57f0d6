"""Adjoint of the ACA recursion at block sizes around its waves and workgroups.

Two clouds, each a leaf of the tree, form the two admissible blocks (n1, n2) and
(n2, n1): fewer rows than a wave, one more than a wave, than two waves and than a
workgroup's 256, and several rounds of it. Every gradient against the oracle's
adjoint on the oracle's pivots. Bounds as for the same comparison on whole
suspensions: dF 1e-13 (rounding), dX and dtheta 1e-11 (u / zeta = 1.1e-12 for the
factors of a late term, a few of which add up).
"""
import numpy as np
import pytest
import torch

import paper_2505_08174_amd as hh
import workloads as wl
from oracle import grad as OG
from oracle import hmatvec as OH
from test_gpu_backward import _maxrel, _oracle_pivots, _rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2", [(3, 65), (64, 257), (129, 1), (300, 40), (530, 300)])
def test_two_clouds(n1, n2):
    from gpu_common import ctx, dev, kernels, say
    say("adjoint", n1, n2)
    rng = np.random.default_rng(n1)
    A, B = wl.lattice_cube(n1, 0.15, seed=1), wl.lattice_cube(n2, 0.15, seed=2)
    A, B = A - A.min(0), B - B.min(0)
    L = 4.0 * max(A.max(), B.max())
    X = np.concatenate([A, B + L])[rng.permutation(n1 + n2)]
    n = n1 + n2
    F, w = wl.normal_forces(n, seed=5), wl.normal_forces(n, seed=6)
    c_leaf = max(n1, n2)
    ko, kg = kernels("mlp")
    ref = OH.build(X, ko, c_leaf, 1.0, 1e-4, 48, pivot="determinant")
    rank, fb, pi, pj = _oracle_pivots(ref)
    assert len(ref.blocks) == 2 and fb.sum() == 0
    tree = hh.build_tree(ctx(), dev(X), c_leaf)
    part = hh.partition(ctx(), tree, 1.0)
    assert np.array_equal(part.export()[0], np.asarray(ref.G))
    lr = hh.aca_build_pivots(ctx(), tree, part, kg, "fp64", rank, fb, pi, pj)
    dF, dX, dth = hh.matvec_backward(ctx(), tree, part, lr, kg, dev(F, torch.float64),
                                     dev(w, torch.float64), "fp64")
    rF, rX, rW, rb = OG.hmatvec_grad(ref, X, F, w, ko)
    eF = _maxrel(dF.cpu().numpy(), rF)
    eX = _rel(dX.cpu().numpy(), rX), _maxrel(dX.cpu().numpy(), rX)
    et = _rel(dth.cpu().numpy(), hh.pack_mlp((rW, rb)))
    say("ranks", rank.tolist(), "dF", eF, "dX", eX, "dtheta", et)
    assert eF < 1e-13 and max(eX) < 1e-11 and et < 1e-11
