"""GPU parity of the update's blur at the sizes where its forms meet.

A lattice is blurred whole in LDS (several features a workgroup up to 48 cells, one up to
about 140), line by line in LDS up to about 1,000 cells, or through memory beyond; within
LDS a pass writes d = min(r, E - 1) + 1 slots below its input or on the other half of its
line, whichever is smaller. Edges and half-widths here lie on both sides of each line; the
result must agree with the oracle bit for bit (fp32 running sums in the same order).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_24067_amd.som as som
import synth
from parity import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("E,r,V,N,chunk", [
    (1, 3, 70, 50, 0), (2, 1, 70, 50, 0), (7, 2, 65, 90, 9), (21, 1, 20, 400, 2), (31, 8, 9, 900, 0),
    (33, 40, 7, 900, 0), (63, 1, 5, 2000, 0), (64, 7, 5, 2000, 2), (64, 63, 5, 2000, 1), (65, 8, 5, 3000, 0),
    (100, 12, 4, 3000, 0), (128, 64, 3, 3000, 1), (139, 139, 2, 3000, 0), (140, 70, 2, 3000, 0), (150, 3, 2, 3000, 0),
    (190, 1, 2, 3000, 0), (200, 5, 3, 9000, 1), (40, 4, 9, 900, 0),
    (41, 5, 9, 900, 0), (20, 6, 9, 900, 0), (201, 7, 2, 3000, 0), (202, 8, 2, 3000, 0), (203, 9, 2, 3000, 0),
    (5, 8, 9, 900, 0), (300, 2, 2, 9000, 0), (300, 6, 2, 9000, 0), (256, 3, 2, 9000, 0), (257, 128, 2, 9000, 0), (320, 40, 2, 9000, 0),
    # lattices that share a workgroup (one for every 512 features), the last workgroup's share ragged, with and
    # without places left out between them
    (1, 2, 1100, 9000, 0), (2, 1, 70001, 9000, 0), (3, 2, 44003, 9000, 0), (5, 3, 27001, 9000, 0),
    (12, 6, 11003, 9000, 0), (16, 8, 8203, 20000, 0), (20, 15, 6203, 20000, 0), (21, 1, 3100, 20000, 0),
    (24, 2, 2777, 20000, 0), (33, 2, 1601, 20000, 0), (41, 2, 1603, 20000, 0), (48, 3, 1111, 20000, 0),
    (48, 24, 1025, 20000, 400), (49, 24, 3, 900, 0),
    (515, 2, 1, 9000, 0), (600, 300, 1, 9000, 0), (700, 400, 1, 9000, 0), (1024, 1, 1, 9000, 0),
])
def test_every_form_of_the_blur(dev, E, r, V, N, chunk, dtype):
    rp, ci = synth.make_csr(700 + E, N, V, lam=2.0)
    W = synth.codebook(700 + E, synth.UNIFORM, V, E * E).astype(dtype)
    rng = np.random.default_rng(E + r)
    bmu = rng.integers(0, E * E, N).astype(np.int32)
    bmu[: N // 2] = rng.integers(0, max(1, E * E // 3))  # one crowded unit: sums past 2^24 at wide windows
    Wd = to_dev(W, dev)
    som.update(Wd, to_dev(rp, dev), to_dev(ci, dev), to_dev(bmu, dev), V, E, r, nnz=len(ci), chunk_features=chunk)
    ref = oracle.update(W.astype(np.float32), E, rp, ci, bmu, r)
    if dtype == np.float16:
        kept = ref == W.astype(np.float32)
        ref = np.where(kept, W.astype(np.float32), ref).astype(np.float16)
    got = Wd.cpu().numpy()
    bad = np.flatnonzero(got != ref)
    assert bad.size == 0, f"{bad.size} of {ref.size} weights differ, first {bad[:5]}"
