"""The large-batch backward pass takes keys in batches by their number of occurrences: batches of one class or of all, of one to
eight handfuls, whole and ragged ones, frequent keys that are neighbours, bag lengths on both sides of the reciprocals that are
kept.  Against one Adagrad step in double."""
import os
import re

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2204_04903_amd", "csrc")
LENGTHS = [1, 2, 3, 4, 5, 8, 9, 30, 255, 256, 257, 1100, 2048, 2500]
BAGS = [1, 2, 511, 512, 513, 40]                           # of the field that pools by the mean
LEAST = 340_000                                            # IDs that a launch in batches has, and more


def constant(name):
    """A constant of the rule that chooses batches."""
    text = open(os.path.join(CSRC, "pk_internal.h")).read()
    a, b = re.search(r"\b" + name + r" = (\d+)(?: << (\d+))?[,;]", text).groups()
    return int(a) << int(b or 0)


def counts_of(kind, n, rng):
    if kind == "ones":
        return np.ones(n, np.int64)
    if kind == "few":
        return rng.integers(2, 9, n)
    if kind == "teams":
        return rng.integers(9, 60, n)
    if kind == "runs":                                     # frequent keys side by side, with others between
        return np.where(np.arange(n) % 250 < 200, 1, rng.integers(9, 257, n))
    c = np.where(rng.random(n) < 0.6, 1, rng.integers(1, 12, n))
    c[rng.permutation(n)[:len(LENGTHS)]] = LENGTHS[:n]
    return c


# handfuls: how many keys a batch holds, in lane groups of a wavefront
@pytest.mark.parametrize("dim,dtype,handfuls", [(2, 0, 1), (3, 1, 1), (6, 0, 1), (10, 1, 1), (32, 0, 2), (64, 0, 4), (100, 0, 8), (200, 1, 8)])
@pytest.mark.parametrize("kind,n", [("ones", 1), ("ones", 513), ("few", 65), ("teams", 63), ("all", 16), ("all", 1100),
                                    ("ones", LEAST + 3), ("few", 75_001), ("teams", 11_111), ("runs", 20_011), ("all", 115_000)])
def test_batches_of_keys(kind, n, dim, dtype, handfuls):
    check(kind, n, dim, dtype, handfuls)


# more IDs, larger batches
@pytest.mark.parametrize("kind,n,dim,dtype,handfuls", [("all", 480_001, 10, 1, 2), ("ones", 1_400_003, 20, 0, 3), ("all", 900_001, 6, 0, 2),
                                                       ("all", 700_001, 64, 1, 8)])
def test_batches_grow_with_the_ids(kind, n, dim, dtype, handfuls):
    check(kind, n, dim, dtype, handfuls)


def check(kind, n, dim, dtype, handfuls):
    from paper_2204_04903_amd.layer import PackedEmbedding
    rng = np.random.default_rng(9800 + 7 * dim + n)
    lr, eps, B = 0.05, 1e-8, 900
    counts = counts_of(kind, n, rng)
    nnz = max(LEAST, int(counts.sum()))
    counts[rng.integers(n)] += nnz - counts.sum()          # (where they are few, one key has what a launch in batches needs)
    rows = 3 * max(n, nnz // 3) + 1
    keys = np.sort(rng.permutation(rows)[:n])
    # sum and mean pooling of one table: its entries carry bag lengths; a wide table that has no occurrence, so that the launch is
    # one in batches whatever the other's dimension
    wide_dim = 48
    fields = [(0, 0), (0, 1), (1, 0)]
    # that it is, and how many handfuls a batch has (the rule goes by the rows that equal fields' IDs can be)
    most = 2 * nnz // 3 + 2
    groups = 64 >> max(0, (dim - 1).bit_length() - 2)
    size = min(64, 8 * groups, max(16, groups, (most // constant("kKeyBatches") + groups // 2) // groups * groups))
    assert nnz >= constant("kBatchNnz") and 16 * most >= 7 * nnz and size == handfuls * groups
    occ = rng.permutation(np.repeat(keys, counts))
    mean = np.resize(BAGS, B)
    mean[np.cumsum(mean) > nnz // 2] = 0
    cuts = np.sort(rng.integers(0, nnz - mean.sum() + 1, B - 1))
    lens = np.concatenate([np.diff(cuts, prepend=0, append=nnz - mean.sum()), mean, np.zeros(B, np.int64)])
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    bag = np.repeat(np.arange(3 * B), lens)
    if kind in ("ones", "all") and n > 100_000:              # keys of one occurrence, and others, in bags on both sides of 512
        alone = np.isin(occ, keys[counts == 1])
        for some in (alone, ~alone) if kind == "all" else (alone,):
            assert set(BAGS) <= set(lens[bag[some & (bag >= B)]])
    cols = 2 * dim + wide_dim
    grad = rng.standard_normal((B, cols), dtype=np.float32)
    gen = torch.Generator("cuda").manual_seed(dim + n)
    layer = PackedEmbedding([(rows, dim, dtype), (2, wide_dim, 0)], fields, debug=2)
    try:
        W, A = layer.table_view(0), layer.acc_view(0)
        W.copy_(torch.randn((rows, dim), device="cuda", generator=gen) * 0.1)
        A.uniform_(0.05, 1.0, generator=gen)
        w, a = W.float().clone(), A.clone()
        wide = torch.full((B, cols + 5), 1e9, device="cuda")             # padded gradient rows
        wide[:, :cols] = torch.from_numpy(grad)
        layer.forward(torch.from_numpy(occ).cuda(), torch.from_numpy(offsets).cuda(), B)
        layer.backward_update(wide[:, :cols] if n % 2 else torch.from_numpy(grad).cuda(), lr, eps)
        assert layer.error_word() == 0
        got_w, got_a = W.float().clone(), A.clone()
    finally:
        layer.close()
    touched = np.sort(keys)
    at = torch.from_numpy(touched).cuda()
    untouched = torch.ones(rows, dtype=torch.bool, device="cuda")
    untouched[at] = False
    assert torch.equal(got_w[untouched], w[untouched]) and torch.equal(got_a[untouched], a[untouched])
    order = np.argsort(occ, kind="stable")
    of = bag[order]
    scale = np.where(of < B, 1.0, 1.0 / np.maximum(lens[of], 1))
    g = np.where((of < B)[:, None], grad[of % B, :dim], grad[of % B, dim:2 * dim]) * scale[:, None]
    first = np.searchsorted(occ[order], touched)
    s = np.add.reduceat(g, first, axis=0)
    w, a, got_w, got_a = (x[at].double().cpu().numpy() for x in (w, a, got_w, got_a))
    ref_a = a + s * s
    ref_w = w - lr * s / (np.sqrt(ref_a) + eps)
    # the sum is rounded to fp32, its square and the accumulator again; a weight takes a few roundings of a step of at most lr
    # in size, and of itself, to 24 or to 8 bits (half a step of 8 bits: up to 2^-8 of the weight, at a power of two)
    assert (np.abs(got_a - ref_a) <= 8 * 2.0 ** -24 * ref_a).all()
    half = 2.0 ** -24 if dtype == 0 else 2.0 ** -8
    assert (np.abs(got_w - ref_w) <= 16 * 2.0 ** -24 * (lr + np.abs(ref_w)) + half * 1.01 * np.abs(ref_w)).all()
