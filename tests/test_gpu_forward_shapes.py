"""Where the forward pass changes its way: bags and fields at the edges of the pooling's runs, rounds and sequence
fields; small batches at every cut of their tables into slices; Partition with chunks longer than one step.
Against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pk_oracle as orc
from test_gpu_parity import run_dense_case
from test_gpu_partition import check_partition

pytestmark = pytest.mark.gpu


def _problem(rng, tables, lens, B):
    """One field per table; lens: [fields, B]."""
    ids = [rng.integers(0, rows, size=int(n.sum())) for (rows, _, _), n in zip(tables, lens)]
    offsets = np.zeros(len(tables) * B + 1, np.int32)
    offsets[1:] = np.cumsum(np.concatenate(lens))
    Wt = []
    for rows, d, dt in tables:
        w = (rng.standard_normal((rows, d)) * 0.01).astype(np.float32)       # bags of 64 and more: the band's |w|
        Wt.append((w.view(np.uint32) >> np.uint32(16)).astype(np.uint16) if dt == 1 else w)
    d_out = sum(d for _, d, _ in tables)
    return dict(tables=tables, B=B, ids=np.concatenate(ids).astype(np.int64), offsets=offsets, Wt=Wt,
                grad=rng.standard_normal((B, d_out)).astype(np.float32), D_out=d_out)


@pytest.mark.parametrize("debug", [0, 2])            # the one-launch forward pass, and the large-batch kernels
@pytest.mark.parametrize("B", [1, 7, 8, 9, 63, 65, 129])
@pytest.mark.parametrize("dim,dtype", [(2, 0), (5, 1), (64, 0), (130, 1), (256, 0)])
def test_runs_and_sequence_fields(B, dim, dtype, debug):
    rng = np.random.default_rng(1000 + 10 * B + dim)
    half = np.where(np.arange(B) % 2 == 0, 0, 127)                        # empty bags first, 63 or 64 on average
    lens = [np.ones(B, int), np.zeros(B, int), rng.integers(0, 3, B), rng.integers(0, 12, B), np.full(B, 63),
            np.full(B, 64), np.full(B, 65), half, np.where(np.arange(B) % 8 == 0, 640, 0)]
    # (no bag above 1000 IDs: the 1e-6 of the band is derived for fp32 sums of up to 1000 terms of about 0.01)
    tables = [(40 + 17 * f, dim, dtype) for f in range(len(lens))]
    run_dense_case(f"runs B={B} dim={dim} dtype={dtype} debug={debug}", tables, [(f, f % 2) for f in range(len(lens))],
                   [_problem(rng, tables, lens, B)], lr=0.01, out_pad=1, debug=debug)


@pytest.mark.parametrize("rows", [3, 1025, 70_000])
@pytest.mark.parametrize("per_table", [0, 1, 1024, 1025, 2048, 2049, 4097, 8193, 16385, 32769, 40_000])
def test_small_batches_at_every_cut(rows, per_table):
    rng = np.random.default_rng(2000 + rows + per_table)
    B, tables = 113, [(rows, 4, 0), (rows + 1, 12, 0)]
    lens = [rng.multinomial(per_table, np.full(B, 1.0 / B)) for _ in tables]
    run_dense_case(f"cut rows={rows} per_table={per_table}", tables, [(0, 1), (1, 0)], [_problem(rng, tables, lens, B)], lr=0.01)


def test_partition_with_chunks_of_several_steps():
    from paper_2204_04903_amd.layer import PackedEmbedding
    rng = np.random.default_rng(3000)
    tables, fields, B = [(1_300_000, 1, 0)], [(0, 0)], 1_100_003          # over 1024 chunks of 1024 distinct keys
    layer = PackedEmbedding(tables, fields)
    try:
        ids = rng.permutation(1_300_000)[:B].astype(np.int64)
        offsets = np.arange(B + 1, dtype=np.int32)
        layer.forward(torch.from_numpy(ids).cuda(), torch.from_numpy(offsets).cuda(), B)
        torch.cuda.synchronize()
        check_partition(layer, orc.plan(tables, fields), [np.sort(ids).astype(np.uint64)], (1, 5, 64))
    finally:
        layer.close()
