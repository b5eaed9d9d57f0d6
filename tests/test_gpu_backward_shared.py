"""FP32 backward in two threads, each with its own context, stream and factors, on one
tree and partition whose first backward these are: the gradients of a backward alone.

dF is summed in a fixed order (equal bits); dX and dtheta add FP32 sums by atomics and
by FP64 slots (1e-12 of the largest covers another order of at most 1e4 FP64 additions).
"""
import threading

import pytest
import torch

import paper_2505_08174_amd as hh
import workloads as wl

pytestmark = pytest.mark.gpu


def _grad(c, t, p, X, F, dU):
    k = hh.Kernel.mlp(c, wl.mlp_weights(1))
    lr = hh.aca_build(c, t, p, k, "fp32", 1e-4)
    g = hh.matvec_backward(c, t, p, lr, k, F, dU, "fp32")
    c.synchronize()
    return [x.cpu() for x in g]


@pytest.mark.parametrize("n,c_leaf", [(700, 33), (1501, 64)])
def test_one_tree_in_two_threads(n, c_leaf):
    from gpu_common import dev, say
    say("backward on a shared tree", n, c_leaf)
    X = dev(wl.lattice_cube(n, 0.1, seed=n))
    F = dev(wl.normal_forces(n, seed=1), torch.float32)
    dU = dev(wl.normal_forces(n, seed=2), torch.float32)
    c0 = hh.Context(0)
    t0 = hh.build_tree(c0, X, c_leaf)
    want = _grad(c0, t0, hh.partition(c0, t0), X, F, dU)
    t = hh.build_tree(c0, X, c_leaf)
    p = hh.partition(c0, t)
    torch.cuda.synchronize()
    got, gate = {}, threading.Barrier(2)

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            c = hh.Context(0)
            gate.wait()
            got[i] = _grad(c, t, p, X, F, dU)

    th = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for x in th:
        x.start()
    for x in th:
        x.join()
    for i in range(2):
        assert torch.equal(got[i][0], want[0]), i
        for a, b in zip(got[i][1:], want[1:]):
            assert (a - b).abs().max() <= 1e-12 * b.abs().max(), i
