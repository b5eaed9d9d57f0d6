"""Kept device blocks when memory runs out: a step whose factors do not fit beside the
kept blocks of another step gets them back, from its own stream and from a context on
another stream, and gives the same bits as before."""
import gc

import pytest
import torch

import paper_2505_08174_amd as hh
import workloads as wl

pytestmark = pytest.mark.gpu


def _step(ctx, n):
    X = torch.tensor(wl.lattice_cube(n, 0.2, seed=n), dtype=torch.float64, device="cuda:0")
    F = torch.tensor(wl.normal_forces(n, seed=n), dtype=torch.float32, device="cuda:0")
    return hh.hmatvec(ctx, X, F, hh.Kernel.rpy(ctx), 64, 1.0, 1e-4, "fp32")


@pytest.mark.parametrize("other_stream", [False, True])
def test_kept_blocks_are_given_back(other_stream):
    from gpu_common import say
    say("kept blocks", other_stream)
    gc.collect()
    ctx = hh.Context(0)
    want = _step(ctx, 20000).cpu()
    with torch.cuda.stream(torch.cuda.Stream()):
        c2 = hh.Context(0) if other_stream else ctx
        _step(c2, 40000)          # its blocks are kept now, several GiB
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free0 = torch.cuda.mem_get_info()[0]
    # leave too little beside the kept blocks for the factors of the next size
    fill, left = [], 1 << 30
    while free0 - left > 0:
        take = min(free0 - left, 64 << 30)
        fill.append(torch.empty(take, dtype=torch.uint8, device="cuda:0"))
        free0 -= take
    try:
        _step(ctx, 33000)
        assert torch.equal(_step(ctx, 20000).cpu(), want)
    finally:
        del fill
        torch.cuda.empty_cache()
