"""Stored products from 131,009 rows on (256 compute units), where one kernel adds the far
field, the near-field rows and the self term and writes the result.

Against the streamed product of the same blocks (other kernels; the factors are the same
bits): in FP32 the results are FP64 sums rounded once, so two roundings apart, 2^-23 of
the largest; with FP64 results the order of the sums differs, n 2^-53 times the sum of the
terms' magnitudes (below 300 times the largest result with random forces): 5e-9.
Against the dense sum: rows of one leaf whose admissible blocks, at all levels, are made
fallbacks and so evaluated entry by entry; the same 5e-9.
"""
import numpy as np
import pytest
import torch

import paper_2505_08174_amd as hh
import workloads as wl
from oracle import dense as OD

pytestmark = pytest.mark.gpu

N = 131100


def _kernel(c, kind):
    return hh.Kernel.rpy(c) if kind == "rpy" else hh.Kernel.mlp(c, wl.mlp_weights(1))


def _setup(kind, prec, c_leaf, eta, eps):
    from gpu_common import dev
    X = wl.lattice_cube(N, 0.1, seed=1)
    F = wl.normal_forces(N, seed=2)
    Fd = dev(F, torch.float64 if prec == "fp64" else torch.float32)
    c = hh.Context(0)
    c.set_budget(160 << 30)
    t = hh.build_tree(c, dev(X), c_leaf)
    p = hh.partition(c, t, eta)
    k = _kernel(c, kind)
    return X, F, Fd, c, t, p, k, hh.aca_build(c, t, p, k, prec, eps, 10)


# near rows: FP32 where a target has fewer than 256 near sources, else FP64
@pytest.mark.parametrize("kind,prec,c_leaf,eta,eps,fallbacks", [
    ("rpy", "fp64", 64, 1.0, 0.5, False), ("mlp", "fp32", 64, 1.0, 0.1, False),
    ("mlp", "bf16", 64, 1.0, 0.1, None), ("rpy", "fp32", 8, 2.0, 0.5, True),
    ("rpy", "fp64", 8, 2.0, 0.5, None), ("mlp", "fp32", 8, 2.0, 0.5, True),
    ("mlp", "fp64", 8, 2.0, 0.5, True), ("mlp", "fp32", 8, 2.0, 1.0, False)])
def test_against_the_streamed_product(kind, prec, c_leaf, eta, eps, fallbacks):
    from gpu_common import say
    X, F, Fd, c, t, p, k, lr = _setup(kind, prec, c_leaf, eta, eps)
    nf = lr.info()["n_fallback"]
    say("final apply", kind, prec, c_leaf, eta, eps, "fallbacks", nf)
    assert fallbacks is None or fallbacks == (nf > 0)
    U = hh.matvec(c, t, p, lr, k, Fd, prec).double()
    c.set_budget(1 << 28)
    ls = hh.aca_build(c, t, p, k, prec, eps, 10)
    V = hh.matvec(c, t, p, ls, k, Fd, prec).double()
    assert ls.info()["bytes"] == 0 and lr.info()["bytes"] > 0   # streamed, stored
    tol = 2.0 ** -23 if prec == "fp32" else 5e-9
    err = ((U - V).abs().max() / V.abs().max()).item()
    assert err <= tol, err


@pytest.mark.parametrize("kind", ["rpy", "mlp"])
def test_fallback_rows_against_the_dense_sum(kind):
    from gpu_common import kernels, say
    X, F, Fd, c, t, p, k, lr = _setup(kind, "fp64", 16, 1.5, 0.5)
    ex = t.export()
    nodes, perm = ex["nodes"], ex["perm"]
    leaf = int(np.flatnonzero(nodes[:, 2] < 0)[len(nodes) // 5])
    a, b = int(nodes[leaf, 0]), int(nodes[leaf, 1])
    G, _ = p.export()
    on = (nodes[G[:, 0], 0] <= a) & (nodes[G[:, 0], 1] >= b)
    f = lr.export()
    say("final apply, dense rows", kind, "blocks", int(on.sum()), "rows", b - a)
    f["fallback"][on] = 1
    f["rank"][on] = 0
    lp = hh.aca_build_pivots(c, t, p, k, "fp64", f["rank"], f["fallback"], f["piv_i"], f["piv_j"])
    assert lp.info()["n_fallback"] >= on.sum() > 0
    U = hh.matvec(c, t, p, lp, k, Fd, "fp64").cpu().numpy()
    rows = perm[a:b]
    ref = OD.dense_u(X, F, kernels(kind)[0], rows)
    err = np.abs(U[rows] - ref).max() / np.abs(ref).max()
    assert err <= 5e-9, err
