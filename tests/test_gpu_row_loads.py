"""GPU parity where codebook rows start at any element's address.

On maps whose width is no multiple of a vector load's elements, and on codebooks that
start inside a larger array, the sweep's vector loads are unaligned and the last group
of a row is read shifted back to end with it. The widths here put that group at every
offset (around the smallest map that takes vector loads, a strip's end, and the end of
a strip's first half); k/256 weights and values make every distance exact, so units and
distances are compared with the oracle bit for bit.
"""
import numpy as np
import pytest
import torch

import synth
import paper_2608_24067_amd.som as som
from parity import compare, compare2, compare_sf, to_dev

pytestmark = pytest.mark.gpu

N, V = 75, 60


def phases(W, rp, ci, dev, tile, two, values=None):
    """The search in its phases, which always take the planned sweep (a whole search of few rows does not)."""
    V, M = W.shape
    N, nnz = len(rp) - 1, len(ci)
    rp, ci = to_dev(rp, dev), to_dev(ci, dev)
    norms = som.codebook_norms(W, V, M)
    out = tuple(torch.empty(N, dtype=t, device=dev) for t in ((torch.int32, torch.float64) * (2 if two else 1)))
    if values is not None:
        ws = som.alloc_workspace_sf(N, M, V, nnz, dev)
        som.bmu_sf_plan(rp, ci, to_dev(values, dev), V, M, nnz, ws)
        som.bmu_sf_sweep(W, norms, V, M, N, nnz, ws, two_best=two)
        som.bmu_sf_finalize(norms, rp, V, M, nnz, out, ws)
    else:
        ws = som.alloc_workspace2(N, M, V, nnz, dev, tile_samples=tile)
        som.bmu_plan(rp, ci, V, M, nnz, ws, tile_samples=tile)
        if two:
            som.bmu2_sweep(W, norms, V, M, N, nnz, ws, tile_samples=tile)
            som.bmu2_finalize(norms, rp, V, M, nnz, out, ws, tile_samples=tile)
        else:
            som.bmu_sweep(W, norms, V, M, N, nnz, ws, tile_samples=tile)
            som.bmu_finalize(norms, rp, V, M, nnz, *out, ws, tile_samples=tile)
    return tuple(t.cpu().numpy() for t in out)


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("M,start", [(3, 0), (4, 1), (5, 0), (7, 1), (8, 3), (9, 0), (257, 0), (259, 1), (511, 0),
                                     (513, 0), (514, 2), (519, 1), (1024, 1), (1027, 0), (1030, 0)])
def test_any_width_and_start(dev, M, start, dtype, tile):
    rp, ci = synth.make_csr(400 + M, N, V)
    W = synth.codebook(400 + M, synth.QUANTISED, V, M)
    W[:, M // 2] = W[:, M - 1]  # a tie: the lower index wins, the last unit is second
    flat = torch.zeros(start + V * M, dtype=dtype, device=dev)
    flat[start:].copy_(torch.from_numpy(W.reshape(-1)))
    view = flat[start:].view(V, M)
    what = f"M={M} start={start} {dtype} TA={tile}"
    compare(W, rp, ci, *phases(view, rp, ci, dev, tile, False), exact=True, what=what)
    compare2(W, rp, ci, phases(view, rp, ci, dev, tile, True), exact=True, what=what)
    if tile == 8:
        vals = synth.values(400 + M, len(ci), synth.VAL_QUANTISED)
        compare_sf(W, rp, ci, vals, phases(view, rp, ci, dev, 8, True, vals), exact=True, what=what + " real")


def test_overflowing_norms_rank_only_owned_neurons(dev):
    # a non-finite bound sends every neuron of a strip to the fp64 stage; the shifted group's
    # leading elements belong to the group before and must not be ranked twice
    V2, M = 12, 515
    rp, ci = synth.make_csr(9, 40, V2)
    W = np.full((V2, M), 3e19, dtype=np.float32)  # norms overflow fp32, not fp64
    W[:, 513] = 1.0
    W[:, 514] = 2.0
    g = phases(to_dev(W, dev), rp, ci, dev, 8, True)
    assert (g[0] == 513).all() and (g[2] == 514).all()
