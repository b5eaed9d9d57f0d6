"""A context that goes from stream to stream, with handles made on one, used on another
and freed with work queued, next to a second context that stays: the bits of one stream."""
import pytest
import torch

import paper_2505_08174_amd as hh
import workloads as wl

pytestmark = pytest.mark.gpu

SIZES = [700, 1500, 699, 2000]


def _step(c, k, X, F):
    return hh.hmatvec(c, X, F, k, 16, 1.0, 1e-6, "fp64")


def test_moving_between_streams():
    from gpu_common import dev, say
    say("streams")
    data = {n: (dev(wl.lattice_cube(n, 0.1, seed=n)), dev(wl.normal_forces(n, seed=n)))
            for n in SIZES}
    c, still = hh.Context(0), hh.Context(0)
    k, ks = hh.Kernel.rpy(c), hh.Kernel.rpy(still)
    want = {n: _step(c, k, *data[n]).cpu() for n in SIZES}
    torch.cuda.synchronize()
    home = torch.cuda.current_stream()
    streams = [torch.cuda.Stream() for _ in range(3)] + [home]
    for i in range(12):
        n, m = SIZES[i % 4], SIZES[(i + 1) % 4]
        s = streams[i % 4]
        h = hh.HMatrix(c, data[n][0], k, 16, 1.0, 1e-6, "fp64")   # on the stream before
        c.set_stream(s)
        with torch.cuda.stream(s):
            U = h @ data[n][1]
            del h
            V = _step(c, k, *data[m])
        W = _step(still, ks, *data[m])                            # takes kept blocks meanwhile
        torch.cuda.synchronize()
        assert torch.equal(U.cpu(), want[n]) and torch.equal(V.cpu(), want[m]), i
        assert torch.equal(W.cpu(), want[m]), i
