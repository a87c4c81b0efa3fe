"""The large-batch backward pass takes keys in batches by their number of occurrences: batches of one class or of all, whole and
ragged ones, bag lengths on both sides of the reciprocals that are kept.  Against one Adagrad step in double."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

LENGTHS = [1, 2, 3, 4, 5, 8, 9, 30, 255, 256, 257, 1100, 2048, 2500]


def counts_of(kind, n, rng):
    if kind == "ones":
        return np.ones(n, np.int64)
    if kind == "few":
        return rng.integers(2, 9, n)
    if kind == "teams":
        return rng.integers(9, 60, n)
    c = np.where(rng.random(n) < 0.6, 1, rng.integers(1, 12, n))
    c[rng.permutation(n)[:len(LENGTHS)]] = LENGTHS[:n]
    return c


@pytest.mark.parametrize("dim,dtype", [(2, 0), (3, 1), (6, 0), (10, 1), (32, 0), (64, 0), (100, 0), (200, 1)])
@pytest.mark.parametrize("kind,n", [("ones", 1), ("ones", 513), ("few", 65), ("teams", 63), ("all", 16), ("all", 1100)])
def test_batches_of_keys(kind, n, dim, dtype):
    from paper_2204_04903_amd.layer import PackedEmbedding
    rng = np.random.default_rng(9800 + 7 * dim + n)
    lr, eps, rows, B = 0.05, 1e-8, 3 * n + 1, 29
    keys = np.sort(rng.permutation(rows)[:n])
    counts = counts_of(kind, n, rng)
    # sum and mean pooling of one table: its entries carry bag lengths; a wide table that has no occurrence takes the launch
    # to the batches whatever the other's dimension
    wide_dim = 48
    fields = [(0, 0), (0, 1), (1, 0)]
    occ = rng.permutation(np.repeat(keys, counts))
    cuts = np.sort(rng.integers(0, len(occ) + 1, 2 * B - 1))
    cuts[B] = max(cuts[B - 1], len(occ) // 2)              # (a bag may hold a large part of all: more than 512 IDs)
    offsets = np.concatenate([[0], np.sort(cuts), np.full(B + 1, len(occ))]).astype(np.int32)
    bag = np.repeat(np.arange(3 * B), np.diff(offsets))
    w = (rng.standard_normal((rows, dim)) * 0.1).astype(np.float32)
    a = rng.uniform(0.05, 1.0, (rows, dim)).astype(np.float32)
    cols = 2 * dim + wide_dim
    grad = rng.standard_normal((B, cols)).astype(np.float32)
    layer = PackedEmbedding([(rows, dim, dtype), (2, wide_dim, 0)], fields, debug=2)
    try:
        W, A = layer.table_view(0), layer.acc_view(0)
        W.copy_(torch.from_numpy(w))
        A.copy_(torch.from_numpy(a))
        w = W.float().cpu().numpy()
        wide = torch.full((B, cols + 5), 1e9, device="cuda")             # padded gradient rows
        wide[:, :cols] = torch.from_numpy(grad)
        layer.forward(torch.from_numpy(occ).cuda(), torch.from_numpy(offsets).cuda(), B)
        layer.backward_update(wide[:, :cols] if n % 2 else torch.from_numpy(grad).cuda(), lr, eps)
        assert layer.error_word() == 0
        got_w, got_a = W.float().cpu().numpy(), A.cpu().numpy()
    finally:
        layer.close()
    scale = np.where(bag < B, 1.0, 1.0 / np.maximum(np.diff(offsets)[bag], 1))
    g = np.where((bag < B)[:, None], grad[bag % B, :dim], grad[bag % B, dim:2 * dim]).astype(np.float64) * scale[:, None]
    s = np.zeros((rows, dim))
    np.add.at(s, occ, g)
    ref_a = a + s * s
    ref_w = w - lr * s / (np.sqrt(ref_a) + eps)
    untouched = np.setdiff1d(np.arange(rows), keys)
    assert (got_w[untouched] == w[untouched]).all() and (got_a[untouched] == a[untouched]).all()
    # the sum is rounded to fp32, its square and the accumulator again; a weight takes a few roundings of a step of at most lr
    # in size, and of itself, to 24 or to 8 bits (half a step of 8 bits: up to 2^-8 of the weight, at a power of two)
    assert (np.abs(got_a - ref_a) <= 8 * 2.0 ** -24 * ref_a).all()
    half = 2.0 ** -24 if dtype == 0 else 2.0 ** -8
    assert (np.abs(got_w - ref_w) <= 16 * 2.0 ** -24 * (lr + np.abs(ref_w)) + half * 1.01 * np.abs(ref_w)).all()
