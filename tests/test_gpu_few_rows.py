"""GPU parity of searches of a few rows, which run without a plan.

The same call in phases (plan, sweep, finalize) takes the planned sweep, so the two paths
are compared bit for bit: on every form of the search, map widths around vector and strip
edges, rows longer than a wave, empty rows, batches on both sides of the line between the
paths, invalid input and non-finite weights; and with the oracle where distances are exact.
"""
import numpy as np
import pytest
import torch

import paper_2608_24067_amd.som as som
import synth
from parity import compare, compare2, compare_sf, gpu_run, gpu_run2, gpu_run_sf, to_dev

pytestmark = pytest.mark.gpu

V = 300


def batch(N, seed, lengths=(12, 0, 1, 64, 65, 130, 9, 15, 16, 17)):
    rng = np.random.default_rng(seed)
    pick = [np.sort(rng.choice(V, lengths[s % len(lengths)], replace=False)) for s in range(N)]
    rp = np.zeros(N + 1, dtype=np.int32)
    rp[1:] = np.cumsum([len(p) for p in pick])
    return rp, np.concatenate(pick + [np.zeros(0, np.int64)]).astype(np.int32)


def both_paths(W, rp, ci, V, M, two, values=None, nnz=None):
    """(direct, its flags, phases, their flags) on device tensors."""
    N = rp.numel() - 1
    nnz = ci.numel() if nnz is None else nnz
    norms = som.codebook_norms(W, V, M)
    make = som.alloc_workspace_sf if values is not None else som.alloc_workspace2
    ws = make(N, M, V, nnz, W.device)
    types = (torch.int32, torch.float64) * (2 if two else 1)
    a, b = (tuple(torch.full((N,), -7, dtype=t, device=W.device) for t in types) for _ in range(2))
    if values is not None:
        som.bmu_sf_search(W, norms, rp, ci, values, V, M, nnz=nnz, two_best=two, out=a, workspace=ws)
    elif two:
        som.bmu2_search(W, norms, rp, ci, V, M, nnz=nnz, out=a, workspace=ws)
    else:
        som.bmu_search(W, norms, rp, ci, V, M, nnz=nnz, bmu=a[0], dist=a[1], workspace=ws)
    fa = som.input_flags(ws, N, M, V, nnz)
    if values is not None:
        som.bmu_sf_plan(rp, ci, values, V, M, nnz, ws)
        som.bmu_sf_sweep(W, norms, V, M, N, nnz, ws, two_best=two)
        som.bmu_sf_finalize(norms, rp, V, M, nnz, b, ws)
    else:
        som.bmu_plan(rp, ci, V, M, nnz, ws)
        if two:
            som.bmu2_sweep(W, norms, V, M, N, nnz, ws)
            som.bmu2_finalize(norms, rp, V, M, nnz, b, ws)
        else:
            som.bmu_sweep(W, norms, V, M, N, nnz, ws)
            som.bmu_finalize(norms, rp, V, M, nnz, b[0], b[1], ws)
    fb = som.input_flags(ws, N, M, V, nnz)
    return a, fa, b, fb


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("M", [1, 3, 5, 8, 511, 513, 1500, 2047])
@pytest.mark.parametrize("N", [1, 65, 256, 1024, 1025, 4096])
def test_equals_phases_and_oracle(dev, N, M, dtype):
    rp, ci = batch(N, 10 * N + M)
    W = synth.codebook(600 + M, synth.QUANTISED, V, M)
    vals = synth.values(600 + M, len(ci), synth.VAL_QUANTISED)
    Wd, rpd, cid, vd = to_dev(W, dev).to(dtype), to_dev(rp, dev), to_dev(ci, dev), to_dev(vals, dev)
    for values in (None, vd):
        for two in (False, True):
            a, fa, b, fb = both_paths(Wd, rpd, cid, V, M, two, values)
            assert fa == fb == 0
            for x, y in zip(a, b):
                assert torch.equal(x, y), (two, values is not None)
    what = f"N={N} M={M} {dtype}"
    if N > 100:
        return
    b, d, _ = gpu_run(Wd, rp, ci, dev, tile_samples=32)
    compare(W, rp, ci, b, d, exact=True, what=what)
    compare2(W, rp, ci, gpu_run2(Wd, rp, ci, dev, tile_samples=16), exact=True, what=what)
    compare_sf(W, rp, ci, vals, gpu_run_sf(Wd, rp, ci, vals, dev), exact=True, what=what)


@pytest.mark.parametrize("weights", ["continuous", "infinite", "nan", "overflowing norms"])
def test_any_weights_equal_phases(dev, weights):
    M = 1030
    rp, ci = batch(31, 3)
    W = synth.codebook(77, synth.UNIFORM, V, M)
    rng = np.random.default_rng(1)
    if weights == "infinite":
        W[rng.integers(0, V, 40), rng.integers(0, M, 40)] = np.inf
    elif weights == "nan":
        W[rng.integers(0, V, 40), rng.integers(0, M, 40)] = np.nan
    elif weights == "overflowing norms":
        W *= 3e19
    for two in (False, True):
        a, _, b, _ = both_paths(to_dev(W, dev), to_dev(rp, dev), to_dev(ci, dev), V, M, two)
        for x, y in zip(a, b):
            assert np.array_equal(x.cpu().numpy(), y.cpu().numpy(), equal_nan=True)


@pytest.mark.parametrize("how", ["past V", "negative", "repeated", "descending", "decreasing rows", "negative first",
                                 "beyond nnz"])
def test_invalid_input_is_flagged_as_by_the_plan(dev, how):
    M, N = 700, 20
    rp, ci = batch(N, 5, (12,))
    W = to_dev(synth.codebook(78, synth.UNIFORM, V, M), dev)
    nnz, at = len(ci), int(rp[9]) + 5
    if how == "past V":
        ci[at] = V
    elif how == "negative":
        ci[at] = -3
    elif how == "repeated":
        ci[at] = ci[at - 1]
    elif how == "descending":
        ci[at] = ci[at - 2]
    elif how == "decreasing rows":
        rp[9] = rp[7]
    elif how == "negative first":
        rp[0] = -4
    else:
        nnz -= 3
    a, fa, b, fb = both_paths(W, to_dev(rp, dev), to_dev(ci, dev), V, M, True, nnz=nnz)
    assert fa == fb != 0
    keep = np.arange(N) != 9 if how in ("repeated", "descending") else np.arange(N) >= 0
    for x, y in zip(a, b):  # a row with unsorted ids has in-range but unspecified results
        assert np.array_equal(x.cpu().numpy()[keep], y.cpu().numpy()[keep])
    assert bool(((a[0] >= 0) & (a[0] < M)).all())


def test_slice_of_a_larger_batch(dev):
    M = 900
    rp, ci = batch(200, 6)
    W = to_dev(synth.codebook(79, synth.UNIFORM, V, M), dev)
    cut = to_dev(rp[50:91], dev)
    a, fa, b, fb = both_paths(W, cut, to_dev(ci, dev), V, M, False, nnz=int(rp[90] - rp[50]))
    assert fa == fb == 0 and torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def later_phases(W2, rp, ci, V, M, two, ws, nnz, values=None, **kw):
    """A sweep of codebook W2 with the plan that a workspace holds, and the finalize."""
    N = rp.numel() - 1
    norms = som.codebook_norms(W2, V, M)
    out = tuple(torch.full((N,), -7, dtype=t, device=W2.device)
                for t in (torch.int32, torch.float64) * (2 if two else 1))
    if values is not None:
        som.bmu_sf_sweep(W2, norms, V, M, N, nnz, ws, two_best=two, **kw)
        som.bmu_sf_finalize(norms, rp, V, M, nnz, out, ws, **kw)
    elif two:
        som.bmu2_sweep(W2, norms, V, M, N, nnz, ws, **kw)
        som.bmu2_finalize(norms, rp, V, M, nnz, out, ws, **kw)
    else:
        som.bmu_sweep(W2, norms, V, M, N, nnz, ws, **kw)
        som.bmu_finalize(norms, rp, V, M, nnz, out[0], out[1], ws, **kw)
    return out


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("kind,two,tile", [("binary", False, 8), ("binary", True, 8), ("binary", False, 16),
                                           ("binary", True, 16), ("binary", False, 32), ("binary", True, 32),
                                           ("real", False, 8), ("real", True, 8)])
@pytest.mark.parametrize("N,M,input", [(1, 700, ""), (40, 1030, ""), (250, 3, ""), (45, 515, "bad id"),
                                       (45, 515, "bad rows")])
def test_the_search_leaves_its_plan(dev, kind, two, tile, N, M, input, dtype):
    rp, ci = batch(N, 40 + N)
    if input == "bad id":
        ci[int(rp[9]) + 5], ci[int(rp[20])] = V, -1
    elif input == "bad rows":
        rp[9] = rp[7]
    nnz = len(ci)
    W = [to_dev(synth.codebook(90 + k, synth.UNIFORM, V, M), dev).to(dtype) for k in range(2)]
    rp, ci = to_dev(rp, dev), to_dev(ci, dev)
    values = to_dev(synth.values(91, nnz, synth.VAL_QUANTISED), dev) if kind == "real" else None
    kw = {"tile_samples": tile}
    ws = (som.alloc_workspace_sf if values is not None else som.alloc_workspace2)(N, M, V, nnz, dev, **kw)
    norms = som.codebook_norms(W[0], V, M)

    def search(W, norms):
        if values is not None:
            return som.bmu_sf_search(W, norms, rp, ci, values, V, M, nnz=nnz, two_best=two, workspace=ws, **kw)
        return (som.bmu2_search if two else som.bmu_search)(W, norms, rp, ci, V, M, nnz=nnz, workspace=ws, **kw)

    want = search(W[1], som.codebook_norms(W[1], V, M))
    ws.fill_(0x5A)
    first = [t.clone() for t in search(W[0], norms)]
    # the finalize once more, from what the search left
    again = tuple(torch.full_like(t, -7) for t in first)
    if values is not None:
        som.bmu_sf_finalize(norms, rp, V, M, nnz, again, ws, **kw)
    elif two:
        som.bmu2_finalize(norms, rp, V, M, nnz, again, ws, **kw)
    else:
        som.bmu_finalize(norms, rp, V, M, nnz, again[0], again[1], ws, **kw)
    flags = som.input_flags(ws, N, M, V, nnz, **kw)
    got = later_phases(W[1], rp, ci, V, M, two, ws, nnz, values, **kw)
    assert som.input_flags(ws, N, M, V, nnz, **kw) == flags
    for a, b in zip(again, first):
        assert torch.equal(a, b)
    for a, b in zip(got, want):
        assert torch.equal(a, b)
