"""Pooled sums against 64 bits: the error does not grow with the bag, whichever way its field takes (tiles of bags:
rows added up in double; a wavefront per bag: up to eight rows as a tree in fp32, the trees in double; keys from the
workspace or from the IDs)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("debug", [0, 2])            # the one-launch forward pass, and the large-batch kernels
@pytest.mark.parametrize("dim", [3, 32, 100, 200])
def test_error_of_pooled_sums_does_not_grow_with_the_bag(dim, debug):
    from paper_2204_04903_amd.layer import PackedEmbedding
    rng = np.random.default_rng(4000 + dim)
    B, rows = 101, 3000
    long_bag = np.where(np.arange(B) == 17, 4000, 3)                       # one long bag in a field of short ones
    lens = [np.full(B, 1), rng.integers(0, 12, B), np.full(B, 25), np.full(B, 63), long_bag, np.full(B, 64), np.full(B, 700)]
    fields = [(0, f % 2) for f in range(len(lens))] + [(0, 1), (0, 0)]     # ... and the two last ways with the other pooling
    lens += [long_bag, np.full(B, 700)]
    offsets = np.zeros(len(fields) * B + 1, np.int32)
    offsets[1:] = np.cumsum(np.concatenate(lens))
    ids = rng.integers(0, rows, size=int(offsets[-1])).astype(np.int64)
    w = rng.standard_normal((rows, dim)).astype(np.float32)
    layer = PackedEmbedding([(rows, dim, 0)], fields, debug=debug)
    try:
        layer.load_table(0, w)
        out = layer.forward(torch.from_numpy(ids).cuda(), torch.from_numpy(offsets).cuda(), B).cpu().numpy().astype(np.float64)
        assert layer.error_word() == 0
    finally:
        layer.close()
    for f, (_, pool) in enumerate(fields):
        for b in range(B):
            x = w[ids[offsets[f * B + b]:offsets[f * B + b + 1]]].astype(np.float64)
            n = max(len(x), 1)
            ref, size = x.sum(0), np.abs(x).sum(0)
            # the sums of 64 bits (here and there: n roundings of at most the sum of the absolute values), rounded to 32 bits;
            # mean pooling rounds 1 / n and the product as well; a tree of eight rounds three times on a row's way
            tree = 3 if lens[f].sum() >= 64 * B else 0
            tol = (2.0 * n * 2.0 ** -53 + tree * 2.0 ** -24) * size + (3 if pool else 1) * 2.0 ** -24 * np.abs(ref)
            tol *= 1 + 2.0 ** -20                          # (terms of second order)
            if pool:
                ref, tol = ref / n, tol / n
            assert (np.abs(out[b, f * dim:(f + 1) * dim] - ref) <= tol).all(), (dim, debug, f, b)
