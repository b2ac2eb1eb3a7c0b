"""GPU parity: the HIP path through the C ABI against the CPU oracle.

Sizes here finish on the oracle in seconds yet span several tiles, strips and
neuron groups with ragged tails; the full-size workloads are in
test_gpu_fullsize.py. Every input is seeded (synth).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_24067_amd.som as som
import synth
from parity import compare, gpu_run, to_dev

pytestmark = pytest.mark.gpu


def case(seed, N, V, M, kind):
    rp, ci = synth.make_csr(seed, N, V)
    W = synth.codebook(seed, kind, V, M)
    return rp, ci, W


@pytest.mark.parametrize("V,M,kind", [
    (2000, 256, synth.QUANTISED), (300, 1, synth.UNIFORM), (37, 5, synth.UNIFORM),
    (1000, 1029, synth.UNIFORM), (64, 4096, synth.UNIFORM), (30000, 300, synth.UNIFORM),
])
def test_norms_match_oracle_bitwise(dev, V, M, kind):
    # both sides add exact fp64 squares in ascending feature order
    W = synth.codebook(7, kind, V, M)
    n_gpu = som.codebook_norms(to_dev(W, dev), V, M).cpu().numpy()
    n_ref = oracle.norms(W)
    assert np.array_equal(n_gpu, n_ref)


# Maps of up to 16,384 units bring their rows in chunks of 112, three in flight (unless they are a
# few whole batches of 128); up to 32,704 a lane reads 128 rows at a time, beyond that 32. Units and
# rows on both sides of each line.
NORM_SHAPES = [(v, 130) for v in (1, 2, 111, 112, 113, 127, 128, 155, 156, 224, 335, 336, 337, 448, 449, 673, 1280,
                                  1307, 1308, 1408)] + \
              [(v, m) for v in (1, 31, 32, 33, 127, 128, 129, 300) for m in (16384, 16385, 32704, 32705, 40001)]


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("V,M", NORM_SHAPES)
def test_norms_of_every_form_match_oracle_bitwise(dev, V, M, dtype):
    W = synth.codebook(V + M, synth.UNIFORM, V, M).astype(dtype)
    n = som.codebook_norms(to_dev(W, dev), V, M).cpu().numpy()
    assert np.array_equal(n, oracle.norms(W.astype(np.float32)))


def test_tiny_workload_bit_exact(dev):
    # the whole 16x16 workload (10,000 rows, V=2000, k/256): every index and distance exact
    cfg = synth.CONFIGS["tiny"]
    rp, ci, W = case(cfg.seed, cfg.N, cfg.V, cfg.M, cfg.kind)
    b, d, _ = gpu_run(W, rp, ci, dev)
    compare(W, rp, ci, b, d, exact=True, what="tiny")


RAGGED = [
    # (seed, N, V, M, kind): N off tile multiples, M off 4 / 256 / 1024 multiples
    (21, 1, 50, 1, synth.QUANTISED),
    (22, 17, 300, 5, synth.QUANTISED),
    (23, 1000, 2000, 300, synth.QUANTISED),
    (24, 333, 500, 1500, synth.QUANTISED),
    (25, 2049, 1000, 1024, synth.UNIFORM),
    (26, 300, 30000, 4099, synth.UNIFORM),
    (27, 77, 30000, 2048, synth.UNIFORM),
    (28, 520, 4000, 3, synth.UNIFORM),
]


@pytest.mark.parametrize("tile,keep", [(8, False), (16, False), (32, False), (8, True)])
@pytest.mark.parametrize("seed,N,V,M,kind", RAGGED)
def test_ragged_shapes(dev, seed, N, V, M, kind, tile, keep):
    rp, ci, W = case(seed, N, V, M, kind)
    b, d, _ = gpu_run(W, rp, ci, dev, tile_samples=tile, keep_order=keep)
    compare(W, rp, ci, b, d, exact=(kind == synth.QUANTISED), what=f"N={N} V={V} M={M} TA={tile} keep={keep}")


def test_tile_size_order_and_repeat_invariance(dev, rules):
    # each sample's dot is its own ascending fp32 sum, so neither the tile size nor the
    # regrouping of samples can change a bit
    rp, ci, W = case(31, 15000, 3000, 16500, synth.UNIFORM)
    assert all(rules.regroups(15000, 16500, len(ci), t) for t in (8, 16, 32))
    runs = [gpu_run(W, rp, ci, dev, tile_samples=t, keep_order=k)[:2]
            for t, k in ((8, False), (16, False), (32, False), (8, True), (16, True), (32, True), (8, False))]
    for b, d in runs[1:]:
        assert np.array_equal(b, runs[0][0]) and np.array_equal(d, runs[0][1])


def test_permuting_samples_permutes_results(dev):
    rp, ci, W = case(32, 700, 5000, 777, synth.UNIFORM)
    b, d, _ = gpu_run(W, rp, ci, dev)
    perm = np.random.default_rng(0).permutation(len(rp) - 1)
    lens = np.diff(rp)[perm]
    rp2 = np.zeros_like(rp)
    rp2[1:] = np.cumsum(lens)
    ci2 = np.concatenate([ci[rp[r]:rp[r + 1]] for r in perm])
    b2, d2, _ = gpu_run(W, rp2, ci2, dev)
    assert np.array_equal(b2, b[perm]) and np.array_equal(d2, d[perm])


def test_constant_codebook_lowest_index(dev):
    rp, ci, _ = case(33, 500, 800, 1500, synth.UNIFORM)
    W = np.full((800, 1500), 0.25, dtype=np.float32)
    b, d, _ = gpu_run(W, rp, ci, dev)
    nnz = np.diff(rp).astype(np.float64)
    assert (b == 0).all()
    assert np.array_equal(d, nnz * 0.75 ** 2 + (800 - nnz) * 0.25 ** 2)


def test_planted_and_tied_units(dev):
    # a copy of sample s's input at j1 < j2 (different strips and groups): distance 0, lowest index wins
    rp, ci, W = case(34, 200, 3000, 2100, synth.UNIFORM)
    W = W.copy()
    plants = {5: (5, 2097), 77: (1023, 1024), 150: (0, 2099)}
    for s, (j1, j2) in plants.items():
        for j in (j1, j2):
            W[:, j] = 0.0
            W[ci[rp[s]:rp[s + 1]], j] = 1.0
    b, d, _ = gpu_run(W, rp, ci, dev)
    for s, (j1, _) in plants.items():
        assert b[s] == j1 and d[s] == 0.0
    compare(W, rp, ci, b, d, exact=False, what="planted", rows=np.arange(0, 200, 7))


def test_empty_rows_rank_by_norm(dev):
    V, M = 400, 700
    W = synth.codebook(35, synth.UNIFORM, V, M)
    rp = np.array([0, 0, 3, 3, 3], dtype=np.int32)
    ci = np.array([2, 10, 399], dtype=np.int32)
    b, d, n = gpu_run(W, rp, ci, dev)
    for s in (0, 2, 3):
        assert b[s] == int(np.argmin(n)) and d[s] == n.min()
    compare(W, rp, ci, b, d, exact=False, what="empty rows")


def long_rows(seed, N, V, lo, hi):
    # rows of lo..hi sorted distinct ids: a wave's 64 rows then hold more ids than
    # the plan stages in LDS, so the plan reads them from global memory
    rng = np.random.default_rng(seed)
    lens = rng.integers(lo, hi + 1, N)
    rp = np.zeros(N + 1, np.int32)
    np.cumsum(lens, out=rp[1:])
    ci = np.concatenate([np.sort(rng.choice(V, n, replace=False)) for n in lens]).astype(np.int32)
    return rp, ci


@pytest.mark.parametrize("tile,keep", [(8, False), (16, False), (32, True)])
def test_long_rows_plan_from_global_memory(dev, tile, keep):
    from test_gpu_row_loads import phases

    rp, ci = long_rows(141, 300, 600, 30, 70)
    W = synth.codebook(141, synth.QUANTISED, 600, 700)
    b, d, _ = gpu_run(W, rp, ci, dev, tile_samples=tile, keep_order=keep)
    compare(W, rp, ci, b, d, exact=True, what=f"long rows tile {tile}")
    # tiles of 8: so few rows are searched without a plan, unless in phases
    compare(W, rp, ci, *phases(to_dev(W, dev), rp, ci, dev, tile, False), exact=True, what=f"planned, tile {tile}")


def test_long_rows_real_values(dev):
    from parity import compare_sf, gpu_run_sf
    from test_gpu_row_loads import phases

    rp, ci = long_rows(142, 200, 500, 30, 70)
    W = synth.codebook(142, synth.QUANTISED, 500, 300)
    vals = synth.values(142, len(ci), synth.VAL_QUANTISED)
    g = gpu_run_sf(W, rp, ci, vals, dev)
    compare_sf(W, rp, ci, vals, g, exact=True, what="long rows, real values")
    planned = phases(to_dev(W, dev), rp, ci, dev, 8, True, vals)
    compare_sf(W, rp, ci, vals, planned, exact=True, what="long rows, real values, planned")


@pytest.mark.parametrize("two_best", [False, True])
def test_overflowing_fp32_norms(dev, two_best):
    # Weights of 3e19 square beyond the fp32 range: those neurons' fp32 norms, and so the
    # strip's bound, are infinite, which sends the strip's neurons to the exact fp64
    # stage. Strip 1 (neurons 512..599) is all huge; strip 0 has a few huge neurons.
    from parity import compare2, gpu_run2

    rp, ci, W = case(131, 400, 300, 600, synth.QUANTISED)
    W[:, 512:] = 3e19
    W[:40, [3, 77, 300]] = 3e19
    if two_best:
        g = gpu_run2(W, rp, ci, dev)
        compare2(W, rp, ci, g, exact=False, what="overflowing norms, two best")
        assert (g[0] < 512).all() and (g[2] < 512).all()
    else:
        b, d, _ = gpu_run(W, rp, ci, dev)
        compare(W, rp, ci, b, d, exact=False, what="overflowing norms")
        assert (b < 512).all() and not np.isin(b, [3, 77, 300]).any()


def test_single_neuron(dev):
    rp, ci, W = case(36, 100, 300, 1, synth.QUANTISED)
    b, d, _ = gpu_run(W, rp, ci, dev)
    assert (b == 0).all()
    compare(W, rp, ci, b, d, exact=True, what="M=1")


def test_batch_slice_offset_row_ptr(dev):
    # row_ptr starting past 0, col_idx the base of the whole array
    rp, ci, W = case(37, 600, 3000, 900, synth.QUANTISED)
    b, d, _ = gpu_run(W, rp, ci, dev)
    s0, s1 = 101, 437
    bs, ds_, _ = gpu_run(W, rp[s0:s1 + 1], ci, dev)
    assert np.array_equal(bs, b[s0:s1]) and np.array_equal(ds_, d[s0:s1])


def test_phases_equal_search_and_flags_clean(dev):
    rp, ci, W = case(38, 999, 3000, 1111, synth.UNIFORM)
    Wd = to_dev(W, dev)
    rpd, cid = to_dev(rp, dev), to_dev(ci, dev)
    V, M, N, nnz = 3000, 1111, 999, int(rp[-1])
    norms = som.codebook_norms(Wd, V, M)
    b1, d1 = som.bmu_search(Wd, norms, rpd, cid, V, M, nnz=nnz)
    ws = som.alloc_workspace(N, M, V, nnz, dev)
    b2 = torch.empty(N, dtype=torch.int32, device=dev)
    d2 = torch.empty(N, dtype=torch.float64, device=dev)
    som.bmu_plan(rpd, cid, V, M, nnz, ws)
    som.bmu_sweep(Wd, norms, V, M, N, nnz, ws)
    som.bmu_finalize(norms, rpd, V, M, nnz, b2, d2, ws)
    assert som.input_flags(ws, N, M, V, nnz) == 0
    assert torch.equal(b1, b2) and torch.equal(d1, d2)
    # the phases only read what the previous one wrote: a second finalize gives the same results
    b2.fill_(-7)
    d2.fill_(-7.0)
    som.bmu_finalize(norms, rpd, V, M, nnz, b2, d2, ws)
    assert torch.equal(b1, b2) and torch.equal(d1, d2)



@pytest.mark.parametrize("tile,keep", [(8, False), (16, True), (32, False)])
def test_invalid_ids_are_flagged_and_stay_local(dev, tile, keep):
    """Ids outside [0, V), unsorted and repeated ids, with valid row pointers: the plan flags them; an id outside
    [0, V) is left out of the dot products (its row ranks as the row without it; the row's length, its ||x||^2,
    still counts it), and every other valid row's result is that of the clean batch, bit for bit (a row's result
    depends on its own ids only)."""
    V, M, N = 500, 1300, 300
    rp, ci, W = case(41, N, V, M, synth.UNIFORM)
    rows = [list(ci[rp[s]:rp[s + 1]]) for s in range(N)]
    multi = [s for s in range(N) if len(rows[s]) >= 3]
    r_hi, r_neg, r_uns, r_dup = multi[1], multi[40], multi[90], multi[-1]
    bad, clean = [list(r) for r in rows], [list(r) for r in rows]
    bad[r_hi][-1] = V + 5       # past the last feature, still ascending
    clean[r_hi] = rows[r_hi][:-1]
    bad[r_neg][0] = -1          # negative, still ascending
    clean[r_neg] = rows[r_neg][1:]
    bad[r_uns][0], bad[r_uns][1] = rows[r_uns][1], rows[r_uns][0]
    bad[r_dup][1] = rows[r_dup][0]

    def csr(rs):
        ptr = np.zeros(N + 1, np.int32)
        np.cumsum([len(r) for r in rs], out=ptr[1:])
        return ptr, np.array([i for r in rs for i in r], dtype=np.int32)

    rp_bad, ci_bad = csr(bad)
    rp_ok, ci_ok = csr(clean)
    som.validate_csr_host(rp_ok, ci_ok, V)
    with pytest.raises(som.SomError):
        som.validate_csr_host(rp_bad, ci_bad, V)
    Wd = to_dev(W, dev)
    norms = som.codebook_norms(Wd, V, M)
    nnz = int(rp_bad[-1])
    ws = som.alloc_workspace(N, M, V, nnz, dev, tile, keep)
    b, d = som.bmu_search(Wd, norms, to_dev(rp_bad, dev), to_dev(ci_bad, dev), V, M, nnz=nnz, workspace=ws,
                          tile_samples=tile, keep_order=keep)
    flags = som.input_flags(ws, N, M, V, nnz, tile, keep)
    assert flags & som.FLAG_ID_RANGE and flags & som.FLAG_UNSORTED and not flags & som.FLAG_ROW_PTR, hex(flags)
    b_ok, d_ok, _ = gpu_run(Wd, rp_ok, ci_ok, dev, tile_samples=tile, norms=norms, keep_order=keep)
    b, d = b.cpu().numpy(), d.cpu().numpy()
    same = np.setdiff1d(np.arange(N), [r_uns, r_dup, r_hi, r_neg])
    assert np.array_equal(b[same], b_ok[same]) and np.array_equal(d[same], d_ok[same])
    for r in (r_hi, r_neg):  # one id skipped: same unit, distance one more (the id still counts in ||x||^2)
        assert b[r] == b_ok[r] and abs(d[r] - (d_ok[r] + 1.0)) <= 1e-12 * abs(d[r]), (r, d[r], d_ok[r])
    assert ((b >= 0) & (b < M)).all()
    compare(W, rp_ok, ci_ok, b_ok, d_ok, exact=False, what="clean batch")

@pytest.mark.parametrize("tile,keep", [(8, False), (16, True)])
def test_negative_first_offset_reads_as_empty(dev, tile, keep):
    """A row_ptr whose first offset is negative would name ids before col_idx: the validator rejects it, and the
    device reads the batch as empty (no id is read), flags its row pointers and still returns in-range results."""
    V, M, N = 400, 700, 50
    rp, ci, W = case(43, N, V, M, synth.UNIFORM)
    rp_neg = (rp - 2).astype(np.int32)
    with pytest.raises(som.SomError):
        som.validate_csr_host(rp_neg, ci, V)
    Wd = to_dev(W, dev)
    norms = som.codebook_norms(Wd, V, M)
    nnz = int(rp[-1])
    for two in (False, True):
        ws = (som.alloc_workspace2 if two else som.alloc_workspace)(N, M, V, nnz, dev, tile, keep)
        search = som.bmu2_search if two else som.bmu_search
        out = search(Wd, norms, to_dev(rp_neg, dev), to_dev(ci, dev), V, M, nnz=nnz, workspace=ws,
                     tile_samples=tile, keep_order=keep)
        flags = som.input_flags(ws, N, M, V, nnz, tile, keep)
        assert flags & som.FLAG_ROW_PTR, hex(flags)
        b, d = out[0].cpu().numpy(), out[1].cpu().numpy()
        assert ((b >= 0) & (b < M)).all() and np.isfinite(d).all()


@pytest.mark.parametrize("tile,keep", [(8, False), (8, True), (16, False)])
def test_decreasing_row_ptr_reads_as_empty(dev, tile, keep):
    """Row pointers that decrease would let rows overlap ([0, nnz, 0, nnz, ...]: every even row spans the whole
    batch) and multiply the work. They are checked before any row is read: the batch is flagged and searched as if
    every row were empty, so every sample gets the unit of smallest norm, lowest index first, and that norm as its
    distance. The sizes keep even the overlapping walk short."""
    V, M, N = 300, 500, 2000
    rp, ci, W = case(44, N, V, M, synth.UNIFORM)
    nnz = int(rp[-1])
    bad = np.zeros(N + 1, np.int32)
    bad[1::2] = nnz
    with pytest.raises(som.SomError):
        som.validate_csr_host(bad, ci, V)
    Wd = to_dev(W, dev)
    norms = som.codebook_norms(Wd, V, M)
    nrm = norms.cpu().numpy()
    order = np.argsort(nrm, kind="stable")  # ascending norm, lower index first among equal norms
    for two in (False, True):
        ws = (som.alloc_workspace2 if two else som.alloc_workspace)(N, M, V, nnz, dev, tile, keep)
        search = som.bmu2_search if two else som.bmu_search
        out = search(Wd, norms, to_dev(bad, dev), to_dev(ci, dev), V, M, nnz=nnz, workspace=ws,
                     tile_samples=tile, keep_order=keep)
        flags = som.input_flags(ws, N, M, V, nnz, tile, keep)
        assert flags & som.FLAG_ROW_PTR, hex(flags)
        res = [t.cpu().numpy() for t in out]
        assert (res[0] == order[0]).all()
        if two:
            assert (res[2] == order[1]).all()
        assert (res[1] == nrm[order[0]]).all()
        if two:
            assert (res[3] == nrm[order[1]]).all()


@pytest.mark.parametrize("name,rows", [("64", 4096), ("256", 1024), ("512", 256)])
def test_workload_prefix(dev, name, rows):
    # the first rows of a full-size workload (rows are drawn per (seed, row)), full map
    cfg = synth.CONFIGS[name]
    rp, ci = synth.make_csr(cfg.seed, rows, cfg.V)
    W = synth.codebook(cfg.seed, cfg.kind, cfg.V, cfg.M)
    b, d, _ = gpu_run(W, rp, ci, dev)
    sample = np.linspace(0, rows - 1, 24).astype(int)
    compare(W, rp, ci, b, d, exact=False, what=f"{name} prefix", rows=sample, nthreads=16)
