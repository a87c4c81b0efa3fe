"""Small batches of tables that several fields read, and of slices with more occurrences or distinct keys than a block
keeps: fields that are empty, of one ID a bag, ragged; occurrences and keys at the edges of what is kept, against the
oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_parity import run_dense_case

pytestmark = pytest.mark.gpu


def case(rng, rows, table_fields, B, lens_of, ids_of, dim=8):
    """One step over tables of `rows`; table_fields[f] is field f's (table, pooling)."""
    tables = [(r, dim, 0) for r in rows]
    lens = np.stack([lens_of(f) for f in range(len(table_fields))])
    offsets = np.zeros(lens.size + 1, np.int32)
    offsets[1:] = np.cumsum(lens.reshape(-1))
    ids = np.concatenate([ids_of(rows[t], int(lens[f].sum())) for f, (t, _) in enumerate(table_fields)]).astype(np.int64)
    D = dim * len(table_fields)
    return dict(tables=tables, fields=table_fields, B=B, ids=ids, offsets=offsets, D_out=D,
                Wt=[(rng.standard_normal((r, dim)) * 0.1).astype(np.float32) for r in rows],
                grad=rng.standard_normal((B, D)).astype(np.float32))


def uniform(rng):
    return lambda rows, n: rng.integers(0, rows, size=n)


@pytest.mark.parametrize("n_fields,n_tables,B", [(2, 1, 1), (3, 1, 682), (3, 1, 683), (26, 2, 64), (13, 3, 300), (40, 3, 97), (1100, 4, 3)])
@pytest.mark.parametrize("mix", ["onehot", "ragged", "empty"])
def test_tables_of_several_fields(n_fields, n_tables, B, mix):
    rng = np.random.default_rng(8000 + n_fields + B)
    fields = [(int(rng.integers(0, n_tables)), f % 2) for f in range(n_fields)]

    def lens_of(f):
        if mix == "onehot":
            return np.ones(B, np.int64)
        if mix == "empty" and f % 3 != 1:
            return np.zeros(B, np.int64)
        return rng.integers(0, 4, size=B)
    pr = case(rng, [3000] * n_tables, fields, B, lens_of, uniform(rng))
    run_dense_case(f"shared {n_fields} {n_tables} {B} {mix}", pr["tables"], fields, [pr], lr=0.01)


@pytest.mark.parametrize("n_fields", [1, 2])
@pytest.mark.parametrize("n", [2047, 2048, 2049, 8192, 8193, 20000])      # occurrences in one slice, all of other keys
def test_slices_with_more_than_is_kept(n, n_fields):
    # one of the table's slices holds the first n keys (every occurrence another key), the rest a few
    rng = np.random.default_rng(8600 + n)
    B = (n + 500) // n_fields + 1
    rows = 1 << 19

    def ids_of(_, count):
        keys = rng.permutation(n)[:count]
        return np.concatenate([keys, rng.integers(0, rows, size=count - len(keys))])
    for mean_len in (1, 2):
        bags = B // mean_len
        lens = np.ones(bags, np.int64) if mean_len == 1 else rng.integers(0, 2 * mean_len + 1, size=bags)
        pr = case(rng, [rows], [(0, f % 2) for f in range(n_fields)], bags, lambda f: rng.permutation(lens), ids_of, dim=4)
        run_dense_case(f"slices {n} {n_fields} {mean_len}", pr["tables"], pr["fields"], [pr], lr=0.01)
