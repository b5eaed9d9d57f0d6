"""Device blocks kept and reused between handles, contexts and streams.

The products are deterministic, so a step whose buffers are blocks freed by
other steps (of other sizes, of another context, with work still queued on
another stream) gives the same bits as the first step of the process did.
"""
import gc
import threading

import numpy as np
import pytest
import torch

import paper_2505_08174_amd as hh
import workloads as wl

pytestmark = pytest.mark.gpu

SIZES = [700, 1500, 699, 2000, 64, 1501]


def _step(ctx, kern, n):
    X = torch.tensor(wl.lattice_cube(n, 0.1, seed=n), dtype=torch.float64, device="cuda:0")
    F = torch.tensor(wl.normal_forces(n, seed=n), dtype=torch.float64, device="cuda:0")
    return hh.hmatvec(ctx, X, F, kern, 16, 1.0, 1e-6, "fp64")


def test_reused_blocks_give_the_same_bits():
    ctx = hh.Context(0)
    kern = hh.Kernel.rpy(ctx)
    first = {n: _step(ctx, kern, n).cpu() for n in SIZES}
    for n in SIZES[::-1] + SIZES:
        assert torch.equal(_step(ctx, kern, n).cpu(), first[n]), n
    # a second context on the same stream, while and after the first one lives
    for keep in (True, False):
        c2 = hh.Context(0)
        k2 = hh.Kernel.rpy(c2)
        if not keep:
            del kern, ctx
            gc.collect()
        for n in SIZES:
            assert torch.equal(_step(c2, k2, n).cpu(), first[n]), (keep, n)


def test_two_streams_and_threads():
    ctx = hh.Context(0)
    kern = hh.Kernel.rpy(ctx)
    want = {n: _step(ctx, kern, n).cpu() for n in SIZES}
    bad = []

    def work(seed):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            c = hh.Context(0)
            k = hh.Kernel.rpy(c)
            rng = np.random.default_rng(seed)
            for _ in range(12):
                n = int(rng.choice(SIZES))
                U = _step(c, k, n)
                c.synchronize()
                if not torch.equal(U.cpu(), want[n]):
                    bad.append((seed, n))
            del k, c

    threads = [threading.Thread(target=work, args=(s,)) for s in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad
