"""GPU parity of regrouped batches that are planned by ranks, at every tile size.

20,001 rows on 16,400 units lie past the line from which a batch is regrouped and have few
enough tiles for the plan by ranks, which reads its rows through the regrouped positions;
rows of 520 ids among them make tiles that fall back to the merge there. The results must be
those of the order given, bit for bit, and the oracle's on sampled rows (k/256 weights and
values: every distance is exact).
"""
import numpy as np
import pytest
import torch

import paper_2608_24067_amd.som as som
import synth
from parity import compare, compare2, compare_sf, gpu_run, gpu_run2, gpu_run_sf, to_dev

pytestmark = pytest.mark.gpu

N, V, M = 20_001, 700, 16_400
LONG = 997  # every so many rows hold 520 ids


@pytest.fixture(scope="module")
def batch(rules):
    rng = np.random.default_rng(17)
    lengths = np.resize((12, 0, 1, 9, 16, 30, 5, 14, 11, 12), N)
    lengths[::LONG] = 520
    pick = [np.sort(rng.choice(V, n, replace=False)) for n in lengths]
    rp = np.zeros(N + 1, dtype=np.int32)
    rp[1:] = np.cumsum(lengths)
    ci = np.concatenate(pick).astype(np.int32)
    assert all(rules.regroups(N, M, len(ci), t) for t in (8, 16, 32))
    assert 3 * N <= len(ci) <= 32 * N and N <= 8 * 13312  # planned by ranks
    W = synth.codebook(17, synth.QUANTISED, V, M)
    rows = np.unique(np.concatenate([rng.choice(N, 40), np.arange(0, N, 4 * LONG), [N - 1]]))
    return rp, ci, W, rows


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("tile", [8, 16, 32])
def test_binary_rows(dev, batch, tile, dtype):
    rp, ci, W, rows = batch
    Wd = to_dev(W, dev).to(dtype)
    got = gpu_run2(Wd, rp, ci, dev, tile_samples=tile)
    for a, b in zip(got, gpu_run2(Wd, rp, ci, dev, tile_samples=tile, keep_order=True)):
        assert np.array_equal(a, b)
    b, d, _ = gpu_run(Wd, rp, ci, dev, tile_samples=tile)
    assert np.array_equal(b, got[0]) and np.array_equal(d, got[1])
    compare(W, rp, ci, b, d, exact=True, what=f"tile {tile}", rows=rows)
    compare2(W, rp, ci, got, exact=True, what=f"tile {tile}", rows=rows)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_real_valued_rows(dev, batch, dtype):
    rp, ci, W, rows = batch
    vals = synth.values(17, len(ci), synth.VAL_QUANTISED)
    Wd = to_dev(W, dev).to(dtype)
    got = gpu_run_sf(Wd, rp, ci, vals, dev)
    for a, b in zip(got, gpu_run_sf(Wd, rp, ci, vals, dev, keep_order=True)):
        assert np.array_equal(a, b)
    for a, b in zip(got, gpu_run_sf(Wd, rp, ci, vals, dev, two_best=False)):
        assert np.array_equal(a, b)
    compare_sf(W, rp, ci, vals, got, exact=True, what="real-valued", rows=rows)


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("how", ["past V", "negative", "repeated", "descending", "decreasing rows"])
def test_invalid_input(dev, batch, how, tile):
    rp, ci, W, _ = batch
    rp, ci, nnz = rp.copy(), ci.copy(), len(ci)
    for row in (4, LONG, N - 1):  # a short row, one whose tile is merged, and the last tile's
        at = int(rp[row]) + 3 if rp[row] + 3 < rp[row + 1] else int(rp[row + 1]) - 1
        if how == "past V":
            ci[at] = V
        elif how == "negative":
            ci[at] = -3
        elif how == "repeated" and row != N - 1:
            ci[at] = ci[at - 1]
        elif how == "descending" and row != N - 1:
            ci[at] = ci[at - 2]
    if how == "decreasing rows":
        rp[N // 2] = rp[N // 2 - 4] - 1
    Wd = to_dev(W, dev)
    norms = som.codebook_norms(Wd, V, M)
    out = []
    for keep in (False, True):
        ws = som.alloc_workspace2(N, M, V, nnz, dev, tile, keep)
        res = som.bmu2_search(Wd, norms, to_dev(rp, dev), to_dev(ci, dev), V, M, nnz=nnz, workspace=ws,
                              tile_samples=tile, keep_order=keep)
        out.append(([t.cpu().numpy() for t in res], som.input_flags(ws, N, M, V, nnz, tile, keep)))
    want = {"past V": som.FLAG_ID_RANGE, "negative": som.FLAG_ID_RANGE, "repeated": som.FLAG_UNSORTED,
            "descending": som.FLAG_UNSORTED, "decreasing rows": som.FLAG_ROW_PTR}[how]
    assert out[0][1] == out[1][1] == want
    same = np.ones(N, dtype=bool)
    if want == som.FLAG_UNSORTED:  # such rows have in-range but unspecified results
        same[[4, LONG]] = False
    for a, b in zip(out[0][0], out[1][0]):
        assert np.array_equal(a[same], b[same])
    for k in (0, 2):
        assert ((out[0][0][k] >= 0) & (out[0][0][k] < M)).all()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("ids", [12, 130, 250, 500])
def test_few_rows_on_a_large_map_equal_their_phases(dev, rules, ids, dtype):
    """64 rows on 512 x 512 units: without a plan, planned as given, and regrouped, by the rows' length and the
    codebook's type; a finalize and a sweep of their own must read what the search left."""
    n, v, m = 64, 600, 1 << 18
    rng = np.random.default_rng(ids)
    ci = np.concatenate([np.sort(rng.choice(v, ids, replace=False)) for _ in range(n)]).astype(np.int32)
    rp = np.arange(n + 1, dtype=np.int32) * ids
    f16 = dtype is torch.float16
    assert rules.rows_direct(n, m, n * ids, 8, f16) == {12: 1, 130: f16, 250: f16, 500: 0}[ids]
    assert rules.regroups(n, m, n * ids, 8) == (ids == 500)
    g = torch.Generator(device=dev).manual_seed(ids)
    W = torch.rand((v, m), device=dev, generator=g).to(dtype)
    norms = som.codebook_norms(W, v, m)
    rpd, cid, nnz = to_dev(rp, dev), to_dev(ci, dev), n * ids
    ws = som.alloc_workspace(n, m, v, nnz, dev)
    b, d = som.bmu_search(W, norms, rpd, cid, v, m, nnz=nnz, workspace=ws)
    want = som.bmu_search(W, norms, rpd, cid, v, m, nnz=nnz, keep_order=True)
    assert torch.equal(b, want[0]) and torch.equal(d, want[1])

    def finalize():
        b, d = torch.full_like(want[0], -7), torch.full_like(want[1], -7)
        som.bmu_finalize(norms, rpd, v, m, nnz, b, d, ws)
        assert torch.equal(b, want[0]) and torch.equal(d, want[1])

    finalize()
    som.bmu_sweep(W, norms, v, m, n, nnz, ws)
    finalize()
    som.bmu_plan(rpd, cid, v, m, nnz, ws)
    som.bmu_sweep(W, norms, v, m, n, nnz, ws)
    finalize()
