"""Pooling with two bags to a lane group (fields of eight IDs a bag and more, up to 64 columns, batches large enough for it), and wider
rows beside it, against the same bags in batches too small for it: both add a bag's rows up in order, in double, so the outputs are the same bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


# (fields, batch): 4096 tiles of two bags per lane group and more, the last one of a field with one bag, with half of its bags, or full
@pytest.mark.parametrize("dim,dtype,n_fields,B", [(6, 0, 300, 833), (8, 1, 300, 896), (20, 0, 100, 665), (64, 1, 60, 556), (200, 0, 20, 411)])
def test_two_bags_to_a_group(dim, dtype, n_fields, B):
    from paper_2204_04903_amd.layer import PackedEmbedding
    rng = np.random.default_rng(9700 + dim)
    rows, cut = 5000, 37
    lens = rng.integers(0, 23, size=(n_fields, B))
    lens[:, 0], lens[:, -1] = 0, 0                                # (empty ones at both ends of a field)
    lens[3] = np.where(np.arange(B) == B // 2, 1500, 10)          # a long one (with fewer than 64 a bag in a cut: no field of sequences there)
    lens[5], lens[6] = 8, 16                                      # whole rounds
    offsets = np.zeros(n_fields * B + 1, np.int64)
    offsets[1:] = np.cumsum(lens.reshape(-1))
    ids = rng.integers(0, rows, size=int(offsets[-1])).astype(np.int64)
    layer = PackedEmbedding([(rows, dim, dtype)], [(0, f % 2) for f in range(n_fields)], debug=2)
    try:
        layer.W[0].copy_(torch.from_numpy(rng.standard_normal((rows, dim)).astype(np.float32)))
        out = torch.full((B, layer.out_dim), float("nan"), device="cuda")
        layer.forward(torch.from_numpy(ids).cuda(), torch.from_numpy(offsets.astype(np.int32)).cuda(), B, out=out)
        assert layer.error_word() == 0
        for b0 in list(range(0, B, cut))[::5] + [B - cut]:
            b1 = min(b0 + cut, B)
            start, n = offsets[:-1].reshape(n_fields, B)[:, b0:b1].reshape(-1), lens[:, b0:b1].reshape(-1)
            o = np.zeros(n.size + 1, np.int64)
            o[1:] = np.cumsum(n)
            part = ids[np.repeat(start - o[:-1], n) + np.arange(o[-1])]
            ref = layer.forward(torch.from_numpy(part).cuda(), torch.from_numpy(o.astype(np.int32)).cuda(), b1 - b0)
            assert layer.error_word() == 0
            assert torch.equal(out[b0:b1], ref), (dim, b0)
    finally:
        layer.close()
