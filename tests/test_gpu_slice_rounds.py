"""Large-batch slices with more records than are kept: rounds of 4096 keys (8192 where slices have 128 K keys), the records
of later rounds moved to the front, a frequent key in the first or the last round, and more such slices than are listed.
Against numpy: integers exactly, and every occurrence's gradient through a step whose sums are small whole numbers."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

WIDE = (4096 << 16) + 1                                    # rows from which slices have 128 K keys


def _keys(name, rng):
    """Per table: rows, pooling, IDs."""
    once = rng.permutation
    if name == "one record too many":
        return [(5000, 0, once(4097)), (5000, 0, once(4096)), (5000, 1, np.concatenate([once(4096), [7]]))]
    if name == "a round exactly, and one key more":
        return [(60_000, 0, np.concatenate([once(4096), rng.integers(0, 4096, 5000)])),
                (60_000, 0, np.concatenate([once(4097), rng.integers(0, 4097, 5000)])),
                (60_000, 1, np.concatenate([once(8193), rng.integers(0, 8193, 600)]))]
    if name == "frequent key of the first round":
        return [(30_000, 0, np.concatenate([once(12_289), np.zeros(30_000, int)]))]
    if name == "frequent key of the last round":
        return [(30_000, 1, np.concatenate([np.full(30_000, 12_288), once(12_289)]))]
    if name == "low IDs frequent":
        return [(1_000_000, t % 2, (rng.random(60_000) ** 6 * 1_000_000).astype(int)) for t in range(3)]
    if name == "long bags":                               # a bag's length does not fit its records
        return [(20_000, 1, (rng.random(200_000) ** 3 * 20_000).astype(int))]
    if name == "more than are listed":
        return [(600, t % 2, (rng.random(16_384 + t) ** 2 * 600).astype(int)) for t in range(270)]
    if name == "wide: one record too many":
        return [(WIDE, 1, rng.integers(0, 100, 8193)), (WIDE + 7, 0, once(8192))]
    if name == "wide: three rounds":
        return [(WIDE, 1, np.concatenate([once(20_000), np.full(40_000, 19_999), rng.integers(0, 20_000, 30_000)]))]
    if name == "wide: two packs, long bags":
        return [(WIDE, 1, (rng.random(150_000) ** 4 * 90_000).astype(int)), (70_000, 1, rng.integers(0, 70_000, 20_000)),
                (3, 0, rng.integers(0, 3, 9_000))]
    raise KeyError(name)


@pytest.mark.parametrize("name", ["one record too many", "a round exactly, and one key more", "frequent key of the first round",
                                  "frequent key of the last round", "low IDs frequent", "long bags", "more than are listed",
                                  "wide: one record too many", "wide: three rounds", "wide: two packs, long bags"])
def test_rounds_of_keys(name):
    from paper_2204_04903_amd.layer import PackedEmbedding
    rng = np.random.default_rng(sum(map(ord, name)))
    case, B = _keys(name, rng), 6
    wide = name.startswith("wide")
    dims = [(1, 2)[t % 2] if wide else 4 for t in range(len(case))]
    layer = PackedEmbedding([(c[0], d, int(wide)) for c, d in zip(case, dims)], [(t, c[1]) for t, c in enumerate(case)], debug=2)
    try:
        lens = []
        for _, _, ids in case:                            # one bag of nearly half, an empty one, the rest evenly
            n = len(ids)
            parts = np.full(4, (n - n // 2) // 4)
            parts[0] += n - n // 2 - parts.sum()
            lens.append(np.concatenate([[n // 2, 0], parts]))
        offsets = np.zeros(len(case) * B + 1, np.int32)
        offsets[1:] = np.cumsum(np.concatenate(lens))
        d_ids = torch.from_numpy(np.concatenate([c[2] for c in case]).astype(np.int64)).cuda()
        d_off = torch.from_numpy(offsets).cuda()
        for W in layer.W:
            W.zero_()
        grad = rng.integers(-3, 4, size=(B, layer.out_dim)).astype(np.float32)
        for step in range(2):                             # the second call finds the first one's workspace
            layer.forward(d_ids, d_off, B)
            torch.cuda.synchronize()
            assert layer.error_word() == 0
            for p in range(layer.n_packs):
                ctx = layer.ctx(p)
                keys = np.concatenate([layer.table_slot[t][1] + c[2] for t, c in enumerate(case) if layer.table_slot[t][0] == p])
                uq, inv, cnt = np.unique(keys, return_inverse=True, return_counts=True)
                assert np.array_equal(ctx["unique"], uq.astype(np.uint32))
                assert np.array_equal(ctx["inverse"], inv)
                assert np.array_equal(ctx["seg_offsets"], np.concatenate([[0], np.cumsum(cnt)]))
        layer.backward_update(torch.from_numpy(grad).cuda(), 0.5, 1e-8)
        for t, (rows, pool, ids) in enumerate(case):
            bag = np.repeat(np.arange(B), lens[t])
            uq, inv = np.unique(ids, return_inverse=True)
            got = layer.acc_view(t)[torch.from_numpy(uq).cuda()].cpu().numpy().astype(np.float64)
            for d in range(dims[t]):
                w = grad[bag, layer.field_col[t] + d].astype(np.float64)
                if pool:
                    w = w / lens[t][bag]
                g = np.bincount(inv, weights=w, minlength=len(uq))
                # sum pooling: whole numbers, g * g exact below 2^24; mean: fp64 sums rounded once to fp32, then squared
                tol = 3.0 * 2.0 ** -24 * g * g + (1e-18 if pool else 0.0)
                assert np.all(np.abs(got[:, d] - g * g) <= tol), (t, d)
    finally:
        layer.close()
