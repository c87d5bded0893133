"""Deposits under graph capture, on the binned path at small sides, and the
path that each of them takes."""
import numpy as np
import pytest
import torch

import oracle
import synthetic
from paper_2110_00328_amd import api

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def uniform(n, count, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return n * torch.rand((count, 3), generator=g, device=DEV).clamp_max(1 - 2.0 ** -24)


def captured(mg, stream, pos, out):
    graph = torch.cuda.CUDAGraph()
    stream.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        mg.cic(pos, out=out)
    return graph


# a graph captured from a deposit still runs after larger deposits on the same
# context have needed larger buffers, and after other memory has been taken
@pytest.mark.parametrize("n", [64, 66])
def test_captured_deposit_outlives_larger_ones(n, monkeypatch):
    monkeypatch.setenv("MGGPU_CIC_DIRECT", "0")
    stream = torch.cuda.Stream()
    pos, more = uniform(n, 50001, 1), [uniform(n, c, 2 + c) for c in (60000, 400000, 1500000)]
    with torch.cuda.stream(stream):
        print("captured deposit", n, flush=True)
        mg = api.Context(n, device=DEV, stream=stream)
        want = mg.cic(pos).clone()
        out = torch.empty((n, n, n), device=DEV)
        graph = captured(mg, stream, pos, out)
        refs = []
        for p in more:
            refs.append(mg.cic(p).clone())
            out.fill_(-7.0)
            graph.replay()
            assert torch.equal(out, want)
        taken = [torch.full((1 << 20,), 3, dtype=torch.int32, device=DEV) for _ in range(16)]
        for p, r in zip(more, refs):
            graph.replay()
            assert torch.equal(out, want) and torch.equal(mg.cic(p), r)
        assert all(bool((t == 3).all()) for t in taken)
        mg.close()


# a deposit under capture, where nothing can be allocated, after one of other
# size: fewer particles on any side, more on sides of no multiple of 16
@pytest.mark.parametrize("n,before,count", [(64, 300000, 1000), (66, 300000, 1000),
                                            (66, 1000, 300000), (66, 300000, 700000)])
def test_deposits_of_other_sizes_can_be_captured(n, before, count):
    stream = torch.cuda.Stream()
    first, pos = uniform(n, before, 11), uniform(n, count, 12)
    print("captured deposit of another size", n, before, count, flush=True)
    plain = api.Context(n, device=DEV)
    want = plain.cic(pos)
    plain.close()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        mg = api.Context(n, device=DEV, stream=stream)
        again = mg.cic(first).clone()
        out = torch.empty((n, n, n), device=DEV)
        graph = captured(mg, stream, pos, out)
        for _ in range(3):
            out.fill_(-7.0)
            graph.replay()
            assert torch.equal(out, want)
            assert torch.equal(mg.cic(first), again)
        mg.close()
