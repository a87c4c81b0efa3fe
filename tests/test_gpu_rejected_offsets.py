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
