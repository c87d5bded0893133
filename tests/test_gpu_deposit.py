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


def deposits(n, pos, monkeypatch, modes):
    t, got = torch.from_numpy(pos).to(DEV), []
    for mode in modes:
        if mode:
            monkeypatch.setenv("MGGPU_CIC_DIRECT", mode)
        else:
            monkeypatch.delenv("MGGPU_CIC_DIRECT", raising=False)
        mg = api.Context(n, device=DEV)
        got.append(mg.cic(t).cpu().numpy())
        mg.close()
    return got


# The binned path, which these sides and numbers would not choose, on a
# Zel'dovich grid (runs of about a tile edge), on particles in no order (runs
# of one, thousands a tile: many batches of the tile pass) and on a clump in one
# cell (runs of 64): one tile (16, and 18's thin ones), tiles that are their own
# neighbour's neighbour (32, 34), whole and thin last tiles beyond (48, 50).
# Both paths add the same fixed-point weights: bit for bit the same.
@pytest.mark.parametrize("n", [16, 18, 32, 34, 48, 50])
def test_binned_deposits_of_grids_and_clumps(n, monkeypatch):
    rng = np.random.default_rng(700 + n)
    grid = synthetic.zeldovich_positions(n, n // 2 + 4, seed=n, dtype=np.float32)
    clump = (3.1 + 0.7 * rng.random((30001, 3))).astype(np.float32)
    far = (n - 0.7 + 0.6 * rng.random((5003, 3))).astype(np.float32)  # over the seam's corner
    far[far >= n] = 0.0
    pos = np.concatenate([grid, rng.uniform(0, n, (60777, 3)).astype(np.float32), clump, far])
    pos[:20] = np.float32(n - 1e-4)
    pos[20:40] = 0.0
    pos[40:80, 0] = np.float32(15.5)  # lower cell on a tile's last layer
    pos[80:120, 1] = np.float32(31.6 % n)
    print("binned deposit, grid and clumps", n, flush=True)
    binned, direct = deposits(n, pos, monkeypatch, ("0", "1"))
    assert np.array_equal(binned.view(np.uint32), direct.view(np.uint32))
    ref = oracle.cic(n, pos.astype(np.float64))
    assert np.max(np.abs(binned - ref)) <= 1e-6 * (1 + np.max(np.abs(ref)))


# the path chosen by itself where that is the binned one (test_cic_path's rows)
@pytest.mark.parametrize("n,npart", [(64, 64), (96, 40), (90, 52), (66, 70)])
def test_chosen_path_equals_direct(n, npart, monkeypatch):
    rng = np.random.default_rng(800 + n)
    pos = np.concatenate([synthetic.zeldovich_positions(n, npart, seed=n, dtype=np.float32),
                          rng.uniform(0, n, (3001, 3)).astype(np.float32),
                          (7.1 + 0.7 * rng.random((20001, 3))).astype(np.float32)])
    print("chosen deposit", n, npart, flush=True)
    chosen, direct = deposits(n, pos, monkeypatch, ("", "1"))
    assert np.array_equal(chosen.view(np.uint32), direct.view(np.uint32))
