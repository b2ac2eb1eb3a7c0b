"""The work this library is measured on: calls of its public entry points over the sizes its users have.

A user of the library maps sparse-binary (or real-valued) rows onto a self-organising map: one row at a time in a
service, a few rows, a mini-batch, a shard of an epoch; on maps from 16x16 to 1024x1024, whose codebook is held in
fp32 or fp16; and, when training, recomputes the norms and updates the codebook between searches. Rows follow the
corpus this library is built for: 1 + Poisson(11) ids per row, Zipf(1.1) features. Codebooks are either freshly
initialised (uniform, or k/256 values) or trained (smooth over the lattice, each weight the mean of 0/1 inputs).
"""
from __future__ import annotations

import math

import torch

import paper_2608_24067_amd.som as som

MEAN_IDS = 12.0

# What a case holds:
#   kind      "search" (one best unit), "two_best", "real" (real-valued rows), "noalloc" (one best unit without a
#             workspace), "eval" (norms, then the two best units) or "update" (the batch update)
#   edge, V, N, dtype   the map is edge x edge units over V features; N rows
#   codebook  "uniform", "quantised" (k/256) or "trained"
#   ids       "ranked" (a feature's id is its frequency rank, as in this repository's benchmark) or "shuffled" (ids in
#             no order of frequency, as in a thesaurus)
#   keep_order   search the rows in the order given
#   radius, chunk, spread   update: box half-width, features per pass (0: all), and how the rows' units are spread


def _case(name, kind, edge, V, N, dtype="float32", codebook="uniform", ids="ranked", keep_order=False, **more):
    c = {"kind": kind, "edge": edge, "V": V, "N": N, "dtype": dtype, "codebook": codebook, "ids": ids,
         "keep_order": keep_order, **more}
    return {"name": name, **c} if name else c


def listed():
    return [
        # One document mapped in a service's loop, which must not allocate.
        _case("one_row_64", "noalloc", 64, 30000, 1, codebook="trained"),
        # A handful of documents with their two best units, on a map kept in half precision.
        _case("few_rows_256_f16", "two_best", 256, 30000, 33, dtype="float16", codebook="trained", ids="shuffled"),
        # The smallest workload of this repository's benchmark, in full.
        _case("tiny_16", "search", 16, 2000, 10000, codebook="quantised"),
        # A mini-batch on a map whose width is no multiple of anything; ids without order of frequency.
        _case("minibatch_75", "search", 75, 12007, 30011, codebook="trained", ids="shuffled"),
        # A shard of a first epoch on the benchmark's 64 x 64 map.
        _case("shard_64", "search", 64, 30000, 2000000),
        # Evaluation after an update: the new norms, then the two best units of a held-out set.
        _case("eval_128", "eval", 128, 30000, 300000, codebook="trained"),
        # An odd half-precision map, odd numbers of rows and features.
        _case("odd_255_f16", "search", 255, 20011, 150001, dtype="float16", codebook="trained", ids="shuffled"),
        # Weighted rows (term weights) on a map of a plain, not a binary, size.
        _case("real_100", "real", 100, 30000, 200000, codebook="trained", ids="shuffled"),
        # A mini-batch on the 512 x 512 map: a 31 GB codebook.
        _case("large_512", "search", 512, 30000, 60000),
        # A mini-batch on the largest map, 63 GB in half precision.
        _case("largest_1024_f16", "search", 1024, 30000, 16000, dtype="float16"),
        # The first epoch's update: half the lattice wide, most rows on few units.
        _case("update_64_first", "update", 64, 30000, 2000000, radius=32, chunk=0, spread="crowded"),
        # A late epoch's update of a half-precision 256 x 256 map within a bounded workspace.
        _case("update_256_f16_late", "update", 256, 30000, 500000, dtype="float16", codebook="trained", radius=3,
              chunk=6000, spread="even"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MOST_PAIRS = 1.2e10       # rows x units of a drawn search (the largest listed one has 1.7e10)
MOST_WEIGHTS = 2.0e9      # weights of a drawn codebook (the largest listed one has 3.1e10)
MOST_UPDATE = 1.2e9       # weights of a drawn update (the largest listed one has 2.0e9)


def draw(rng):
    """One more case: any kind, sizes spread over their ranges on a logarithmic scale."""
    group = rng.choice(["few", "search", "search", "two_best", "eval", "real", "update"])
    dtype = rng.choice(["float32", "float16"])
    ids = rng.choice(["ranked", "shuffled"])
    codebook = rng.choice(["uniform", "trained"])
    if group == "update":
        edge = _log_int(rng, 16, 256)
        V = min(_log_int(rng, 1500, 30000), int(MOST_UPDATE / edge ** 2))
        radius = max(1, _log_int(rng, 1, edge // 2))
        chunk = rng.choice([0, 0, max(64, V // 3)])
        return _case(None, "update", edge, V, _log_int(rng, 2000, 1500000), dtype, codebook, ids, radius=radius,
                     chunk=chunk, spread=rng.choice(["even", "crowded"]))
    if group == "few":
        edge = _log_int(rng, 16, 256)
        kind = rng.choice(["noalloc", "search", "two_best"])
        V = min(_log_int(rng, 2000, 30000), int(MOST_WEIGHTS / edge ** 2))
        return _case(None, kind, edge, V, _log_int(rng, 1, 64), "float32" if kind == "noalloc" else dtype, codebook, ids)
    edge = _log_int(rng, 16, 512)
    V = max(1500, min(_log_int(rng, 2000, 30000), int(MOST_WEIGHTS / edge ** 2)))
    N = _log_int(rng, 1000, min(2000000, MOST_PAIRS / edge ** 2))
    return _case(None, group, edge, V, N, dtype, codebook, ids,
                 keep_order=group == "search" and rng.random() < 0.2)


# ------------------------------------------------------------------ inputs


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
    return g


def _zipf(V):
    p = torch.arange(1, V + 1, dtype=torch.float64).pow(-1.1)
    return p / p.sum()


def _names(case, g):
    """The id of every frequency rank (None: the rank itself)."""
    return torch.randperm(case["V"], device="cuda", generator=g) if case["ids"] == "shuffled" else None


def _rows(case, name, g):
    """CSR rows: 1 + Poisson(11) distinct Zipf(1.1) ids each, ascending. Returns (row_ptr, col_idx) int32."""
    V, N = case["V"], case["N"]
    cdf = _zipf(V).cumsum(0).to("cuda")
    counts, cols = [], []
    K = 48  # draws per row; a row keeps its first distinct ones
    for a in range(0, N, 400000):
        n = min(400000, N - a)
        want = 1 + torch.poisson(torch.full((n, 1), 11.0, device="cuda"), generator=g).long()
        u = torch.rand((n, K), dtype=torch.float64, device="cuda", generator=g)
        d = torch.searchsorted(cdf, u).clamp_(max=V - 1)
        s, at = torch.sort(d, dim=1, stable=True)
        first = torch.ones_like(s, dtype=torch.bool)
        first[:, 1:] = s[:, 1:] != s[:, :-1]
        fresh = torch.zeros_like(first).scatter_(1, at, first)  # in the order drawn
        keep = fresh & (fresh.cumsum(1) <= want)
        d = name[d] if name is not None else d
        d = torch.where(keep, d, V).sort(dim=1).values
        ok = d < V
        counts.append(ok.sum(1))
        cols.append(d[ok].int())
    row_ptr = torch.zeros(N + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.cat(counts), 0, out=row_ptr[1:])
    return row_ptr.int(), torch.cat(cols)


def _codebook(case, name, g):
    """V x M weights: uniform in [0, 1), k/256, or as training leaves them: smooth over the lattice, each the mean of 0/1 inputs."""
    V, E = case["V"], case["edge"]
    W = torch.empty((V, E * E), dtype=getattr(torch, case["dtype"]), device="cuda")
    rows = max(1, min(V, (1 << 28) // (E * E)))
    logit = None
    if case["codebook"] == "trained":
        p = (MEAN_IDS * _zipf(V)).clamp(1e-6, 0.8)
        logit = torch.log(p / (1 - p)).float().to("cuda")
        if name is not None:
            logit = torch.empty_like(logit).scatter_(0, name, logit)
    coarse = max(2, E // 8)
    for a in range(0, V, rows):
        n = min(rows, V - a)
        if case["codebook"] == "trained":
            z = torch.randn((n, 1, coarse, coarse), device="cuda", generator=g)
            z = torch.nn.functional.interpolate(z, size=(E, E), mode="bilinear", align_corners=True)
            w = torch.sigmoid(z.view(n, E * E).mul_(2.0).add_(logit[a:a + n, None]))
        else:
            w = torch.rand((n, E * E), device="cuda", generator=g)
            if case["codebook"] == "quantised":
                w = torch.floor(w * 256) / 256
        W[a:a + n].copy_(w)
    return W


def _units(case, g):
    """Each row's unit for an update: spread over the lattice, or most rows on a few units (an untrained map)."""
    N, M = case["N"], case["edge"] ** 2
    u = torch.randint(0, M, (N,), device="cuda", generator=g)
    if case["spread"] == "crowded":
        few = torch.randint(0, M, (8,), device="cuda", generator=g)
        to = few[(torch.rand(N, device="cuda", generator=g).pow(2) * 8).long().clamp_(max=7)]
        u = torch.where(torch.rand(N, device="cuda", generator=g) < 0.8, to, u)
    return u.int()


def prepare(case, seed):
    """What a user's program holds before the call: the batch, the codebook, its norms, and buffers of the right size."""
    g = _generator(seed)
    V, N, E, kind = case["V"], case["N"], case["edge"], case["kind"]
    M = E * E
    name = _names(case, g)
    row_ptr, col_idx = _rows(case, name, g)
    nnz = col_idx.numel()
    st = {"case": case, "row_ptr": row_ptr, "col_idx": col_idx, "nnz": nnz, "W": _codebook(case, name, g)}
    if kind == "update":
        st["bmu"] = _units(case, g)
        st["workspace"] = torch.empty(som.update_workspace_bytes(V, E, N, case["chunk"]), dtype=torch.uint8,
                                      device="cuda")
        return st
    st["norms"] = som.codebook_norms(st["W"], V, M)
    two = kind in ("two_best", "eval")
    st["out"] = tuple(torch.empty(N, dtype=t, device="cuda")
                      for t in ((torch.int32, torch.float64) * (2 if two else 1)))
    if kind == "real":
        st["values"] = 1.0 - torch.rand(nnz, device="cuda", generator=g)  # term weights in (0, 1]
        st["workspace"] = som.alloc_workspace_sf(N, M, V, nnz, "cuda")
    elif two:
        st["workspace"] = som.alloc_workspace2(N, M, V, nnz, "cuda")
    elif kind == "search":
        st["workspace"] = som.alloc_workspace(N, M, V, nnz, "cuda", keep_order=case["keep_order"])
    return st


def run(st):
    """One pass: the search's units and distances, the norms too where they are computed, or the updated codebook."""
    c = st["case"]
    V, M, W, rp, ci, nnz = c["V"], c["edge"] ** 2, st["W"], st["row_ptr"], st["col_idx"], st["nnz"]
    kind = c["kind"]
    if kind == "update":
        return som.update(W, rp, ci, st["bmu"], V, c["edge"], c["radius"], nnz=nnz, chunk_features=c["chunk"],
                          workspace=st["workspace"])
    norms, out = st["norms"], st["out"]
    if kind == "search":
        return som.bmu_search(W, norms, rp, ci, V, M, nnz=nnz, bmu=out[0], dist=out[1], workspace=st["workspace"],
                              keep_order=c["keep_order"])
    if kind == "noalloc":
        return som.bmu_search_noalloc(W, norms, rp, ci, V, M, nnz, out[0], out[1])
    if kind == "real":
        return som.bmu_sf_search(W, norms, rp, ci, st["values"], V, M, nnz=nnz, out=out, workspace=st["workspace"])
    if kind == "eval":
        som.codebook_norms(W, V, M, out=norms)
        return (norms, *som.bmu2_search(W, norms, rp, ci, V, M, nnz=nnz, out=out, workspace=st["workspace"]))
    return som.bmu2_search(W, norms, rp, ci, V, M, nnz=nnz, out=out, workspace=st["workspace"])


def work(case):
    """Each input read once and each output written once; of the codebook, the rows of features that the batch holds."""
    V, N, M = case["V"], case["N"], case["edge"] ** 2
    e = 2 if case["dtype"] == "float16" else 4
    ids = 4.0 * (N + 1) + 4.0 * MEAN_IDS * N
    if case["kind"] == "update":  # the blur is six running sums, two operations each; one division
        return {"bytes": ids + 4.0 * N + float(V) * M * e, "flops": MEAN_IDS * N + float(V) * M * 13}
    p = (MEAN_IDS * _zipf(V)).clamp(max=1.0)
    touched = float((1 - torch.exp(-p * N)).sum())
    two = case["kind"] in ("two_best", "eval")
    rows = float(V) if case["kind"] == "eval" else touched
    real = case["kind"] == "real"
    flops = float(N) * M * (MEAN_IDS * (2 if real else 1) + 2)
    if case["kind"] == "eval":
        flops += 2.0 * V * M
    return {"bytes": rows * M * e + 8.0 * M + ids * (2 if real else 1) + 12.0 * N * (2 if two else 1), "flops": flops}


def tolerance(case):
    """Distances are fp64 over fp32 sums of about 12 terms; units may differ where two are equally near to that precision."""
    if case["kind"] == "update":
        # binary16 storage rounds by 2^-11; fp32 running sums over an unnormalised blur are off by 4e-7 as measured
        return {"rel": 8e-4, "max": 4e-3} if case["dtype"] == "float16" else {"rel": 1e-5, "max": 1e-3}
    if case["codebook"] == "quantised":
        return "exact"  # every sum is a multiple of 2^-16 below 2^15
    return {"rel": 4e-7, "max": 4e-6, "differ": 2e-4}


# ------------------------------------------------------------------ the same in 64 bits


def exact(case, seed):
    """The outputs of run() in 64 bits; None for a unit's index (ties) and for cases too large to compute so."""
    V, N, E = case["V"], case["N"], case["edge"]
    M = E * E
    if case["kind"] == "update":
        if float(V) * M * E > 2e12:
            return None
    elif float(N) * M * MEAN_IDS > 2.5e11 or float(V) * M > 1e10:
        return None
    g = _generator(seed)
    name = _names(case, g)
    rp, ci = _rows(case, name, g)
    W = _codebook(case, name, g)
    if case["kind"] == "update":
        return _exact_update(case, rp.long(), ci.long(), W, _units(case, g))
    real = case["kind"] == "real"
    x = (1.0 - torch.rand(ci.numel(), device="cuda", generator=g)) if real else torch.ones(ci.numel(), device="cuda")
    return _exact_search(case, rp.long(), ci.long(), x.double(), W)


def _exact_search(case, rp, ci, x, W):
    N, M = case["N"], case["edge"] ** 2
    d1 = torch.full((N,), math.inf, dtype=torch.float64, device="cuda")
    d2 = d1.clone()
    lens = rp[1:] - rp[:-1]
    xsq = torch.zeros(N, dtype=torch.float64, device="cuda").index_add_(
        0, torch.repeat_interleave(torch.arange(N, device="cuda"), lens), x * x)
    norms = torch.empty(M, dtype=torch.float64, device="cuda")
    cols = max(1, min(M, (1 << 28) // W.shape[0]))
    for i in range(0, M, cols):
        w = W[:, i:i + cols].double()
        norms[i:i + cols] = (w * w).sum(0)
        rows = max(1, (1 << 27) // w.shape[1])
        for a in range(0, N, rows):
            b = min(N, a + rows)
            p, q = int(rp[a]), int(rp[b])
            dot = torch.nn.functional.embedding_bag(ci[p:q], w, rp[a:b] - p, mode="sum", per_sample_weights=x[p:q])
            d = norms[i:i + cols] - 2 * dot + xsq[a:b, None]
            top = torch.topk(d, min(2, d.shape[1]), dim=1, largest=False).values
            two = torch.cat([d1[a:b, None], d2[a:b, None], top], 1).sort(1).values
            d1[a:b], d2[a:b] = two[:, 0], two[:, 1]
    if case["kind"] == "eval":
        return norms, None, d1, None, d2
    return (None, d1, None, d2) if case["kind"] == "two_best" else (None, d1)


def _exact_update(case, rp, ci, W, bmu):
    N, E, V, r = case["N"], case["edge"], case["V"], case["radius"]
    M = E * E
    at = torch.arange(E, device="cuda")
    box = ((at[:, None] - at[None, :]).abs() <= r).double()
    box3 = box @ box @ box
    near = ((at[:, None] - at[None, :]).abs() <= 3 * r).double()

    def both(m, f):  # m f m^T for every lattice of f
        n = f.shape[0]
        f = (f.reshape(n * E, E) @ m).reshape(n, E, E).transpose(1, 2).reshape(n * E, E)
        return (f @ m).reshape(n, E, E).transpose(1, 2).reshape(n, M)

    unit = bmu.long()
    den = torch.zeros(M, dtype=torch.float64, device="cuda").index_add_(
        0, unit, torch.ones(N, dtype=torch.float64, device="cuda"))
    reached = (both(near, (den > 0).double().view(1, M)) > 0.5).view(M)
    den = both(box3, den.view(1, M)).view(M)
    unit = torch.repeat_interleave(unit, rp[1:] - rp[:-1])
    by, order = torch.sort(ci)
    unit = unit[order]
    out = torch.empty((V, M), dtype=torch.float64, device="cuda")
    rows = max(1, (1 << 27) // M)
    for a in range(0, V, rows):
        n = min(rows, V - a)
        p, q = (int(k) for k in torch.searchsorted(by, torch.tensor([a, a + n], device="cuda")))
        num = torch.zeros(n * M, dtype=torch.float64, device="cuda").index_add_(
            0, (by[p:q] - a) * M + unit[p:q], torch.ones(q - p, dtype=torch.float64, device="cuda"))
        num = both(box3, num.view(n, M))
        out[a:a + n] = torch.where(reached, (num / den).clamp_(0, 1), W[a:a + n].double())
    return out
