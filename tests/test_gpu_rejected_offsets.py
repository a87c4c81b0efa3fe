"""Outputs after rejected offsets have no defined values, but every one is written: finite sums of rows that exist,
never what the output's memory held."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from helpers import small_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("debug", [0, 2])            # the one-launch forward pass, and the large-batch kernels
@pytest.mark.parametrize("place,value", [(3, 14), (3, 0), (5, 10**9), (5, -7), (8, 10**9), (8, 0), (0, 2), (16, 1)])
@pytest.mark.parametrize("dim", [2, 20])
def test_every_output_is_written(place, value, dim, debug):
    from paper_2204_04903_amd.layer import PackedEmbedding
    tables, fields, B = [(50, dim, 0), (31, dim, 0)], [(0, 0), (1, 1)], 8
    pr = small_problem(96, B=B, tables=tables, fields=fields, max_len=3, allow_empty=False)
    bad = pr["offsets"].copy()
    bad[place] = value
    layer = PackedEmbedding(tables, fields, debug=debug)
    try:
        for t in range(len(tables)):
            layer.load_table(t, pr["Wt"][t])
        out = torch.full((B, layer.out_dim), float("nan"), dtype=torch.float32, device="cuda")
        layer.forward(torch.from_numpy(pr["ids"]).cuda(), torch.from_numpy(bad).cuda(), B, out=out)
        torch.cuda.synchronize()
        assert layer.error_word() & 1
        assert torch.isfinite(out).all()
    finally:
        layer.close()


# the pooling with two bags to a lane group (fields of eight IDs a bag and more, batches that have 4096 tiles of such bags):
# (field, bag) of the offset; inside a field, at both ends of one and of all
@pytest.mark.parametrize("place,value", [((10, 300), 3), ((10, 301), 10**9), ((11, 664), -7), ((12, 0), 10**9), ((99, 664), 5),
                                         ((100, 0), 0), ((0, 0), 2), ((0, 1), -2**31)])
def test_every_output_of_pairs_is_written(place, value):
    from paper_2204_04903_amd.layer import PackedEmbedding
    dim, F, B = 20, 100, 665
    tables, fields = [(5000, dim, 0)], [(0, f % 2) for f in range(F)]
    pr = small_problem(97, B=B, tables=tables, fields=fields, max_len=22)
    assert pr["offsets"][-1] >= 8 * F * B
    layer = PackedEmbedding(tables, fields, debug=2)
    try:
        layer.load_table(0, pr["Wt"][0])
        ids, offsets = torch.from_numpy(pr["ids"]).cuda(), torch.from_numpy(pr["offsets"]).cuda()
        layer.forward(ids, offsets, B)                   # (the workspace then holds a batch's offsets and keys)
        assert layer.error_word() == 0
        offsets[place[0] * B + place[1]] = value
        out = torch.full((B, layer.out_dim), float("nan"), dtype=torch.float32, device="cuda")
        layer.forward(ids, offsets, B, out=out)
        torch.cuda.synchronize()
        assert layer.error_word() & 1
        assert torch.isfinite(out).all()
    finally:
        layer.close()
