"""The backward pass handles a key by its number of occurrences: keys at the limits between the ways it takes
(a lane group, a wavefront, one piece, several pieces), for dimensions at the edges of a lane's four columns,
against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_parity import run_dense_case

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 4, 5, 8, 9, 16, 255, 256, 257, 512, 1023, 1024, 1025, 2047, 2048, 2049, 3100, 5000]


@pytest.mark.parametrize("debug", [0, 2])            # the one-launch forward pass, and the large-batch kernels
@pytest.mark.parametrize("dims,dtype", [((1, 3, 4), 0), ((5, 10, 33), 0), ((64, 100, 256), 0), ((3, 6, 64), 1), ((7, 130, 32), 1)])
def test_keys_at_the_limits(dims, dtype, debug):
    rng = np.random.default_rng(900 + sum(dims) + dtype)
    B = 97
    tables = [(150 + 40 * i, d, dtype) for i, d in enumerate(dims)]
    fields = [(0, 0), (1, 1), (2, 1)]
    ids, lens = [], []
    for rows, _, _ in tables:
        keys = rng.permutation(rows)[:len(COUNTS)]
        part = rng.permutation(np.repeat(keys, COUNTS))
        cut = np.sort(rng.integers(0, len(part) + 1, size=B - 1))
        ids.append(part)
        lens.append(np.diff(np.concatenate([[0], cut, [len(part)]])))
    offsets = np.zeros(len(fields) * B + 1, np.int32)
    offsets[1:] = np.cumsum(np.concatenate(lens))
    Wt = []
    for rows, d, dt in tables:
        w = (rng.standard_normal((rows, d)) * 0.1).astype(np.float32)
        Wt.append((w.view(np.uint32) >> np.uint32(16)).astype(np.uint16) if dt == 1 else w)
    step = dict(tables=tables, fields=fields, B=B, ids=np.concatenate(ids).astype(np.int64), offsets=offsets, Wt=Wt,
                grad=rng.standard_normal((B, sum(dims))).astype(np.float32), D_out=sum(dims))
    run_dense_case(f"limits {dims} {dtype} {debug}", tables, fields, [step], lr=0.01, out_pad=3, grad_pad=1, debug=debug)
