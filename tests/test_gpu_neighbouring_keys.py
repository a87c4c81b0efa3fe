"""Neighbouring keys of nine to 256 occurrences, which the backward pass meets in one handful of a wavefront and, for
rows of up to 16 columns, deals to teams of lane groups: from one such key to all of a handful, beside shorter and
longer ones, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_parity import run_dense_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_met", [1, 2, 5, 16, 17, 33, 64, 150])     # neighbouring keys with more than eight occurrences
@pytest.mark.parametrize("dim,dtype,pool", [(1, 0, 0), (2, 1, 1), (3, 0, 1), (4, 0, 0), (8, 1, 0), (16, 0, 1), (17, 0, 0)])
def test_neighbouring_frequent_keys(dim, dtype, pool, n_met):
    rng = np.random.default_rng(7000 + 100 * dim + n_met)
    rows, first = 400, int(rng.integers(0, 70))
    counts = rng.integers(0, 9, size=rows)
    counts[first:first + n_met] = rng.choice([9, 12, 16, 17, 63, 64, 65, 255, 256, 257], size=n_met)
    ids = rng.permutation(np.repeat(np.arange(rows), counts)).astype(np.int64)
    B = 61
    cut = np.sort(rng.integers(0, len(ids) + 1, size=B - 1))
    offsets = np.concatenate([[0], cut, [len(ids)]]).astype(np.int32)
    w = (rng.standard_normal((rows, dim)) * 0.1).astype(np.float32)
    if dtype == 1:
        w = (w.view(np.uint32) >> np.uint32(16)).astype(np.uint16)
    tables, fields = [(rows, dim, dtype)], [(0, pool)]
    step = dict(tables=tables, fields=fields, B=B, ids=ids, offsets=offsets, Wt=[w],
                grad=rng.standard_normal((B, dim)).astype(np.float32), D_out=dim)
    run_dense_case(f"neighbours {dim} {n_met}", tables, fields, [step], lr=0.01)
